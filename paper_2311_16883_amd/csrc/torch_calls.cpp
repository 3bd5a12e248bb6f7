// The single-tensor calls of libbsr_actprune with torch tensors as arguments: what binding.py's
// functions do between Python and the C ABI, in native code.  Argument checks, output and workspace
// tensors (torch's caching allocator), device pointers, the current stream, then one C call with the GIL
// released.  No step of the pruning path is computed here.
//
// Why native: a layer of a training step is three calls of a few microseconds of GPU time each, and
// marshalling in Python took 8 to 10 us a call (torch.cuda.current_stream() 2.9 us, torch.empty 1.4 us
// per output, ctypes 0.6 us and more); here it is about 2 us.
//
// Every function takes positional arguments only (binding.py has the keyword forms and turns a negative
// return value, a BSR_ERR_* code, into an exception).
#include <Python.h>

#include <climits>

#include <ATen/ops/empty.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "bsr_actprune.h"

namespace {

// A Python exception is set already.
struct PythonError {};

[[noreturn]] void value_error(const std::string &what) {
  PyErr_SetString(PyExc_ValueError, what.c_str());
  throw PythonError();
}

const at::Tensor &tensor(PyObject *o, const char *what) {
  if (!THPVariable_Check(o)) {
    PyErr_Format(PyExc_TypeError, "%s must be a tensor, not %s", what, Py_TYPE(o)->tp_name);
    throw PythonError();
  }
  return THPVariable_Unpack(o);
}

int64_t integer(PyObject *o) {
  const long long v = PyLong_AsLongLong(o);
  if (v == -1 && PyErr_Occurred()) throw PythonError();
  return v;
}

// A block extent: beyond the range of int it becomes a value that the library refuses.
int extent(PyObject *o) {
  const int64_t v = integer(o);
  return v > INT_MAX ? INT_MAX : v < 0 ? -1 : (int)v;
}

// int(o)
int64_t converted_integer(PyObject *o) {
  if (PyLong_Check(o)) return integer(o);
  PyObject *n = PyNumber_Long(o);
  if (n == nullptr) throw PythonError();
  const long long v = PyLong_AsLongLong(n);
  Py_DECREF(n);
  if (v == -1 && PyErr_Occurred()) throw PythonError();
  return v;
}

// float(o)
double real(PyObject *o) {
  if (PyFloat_Check(o)) return PyFloat_AS_DOUBLE(o);
  PyObject *f = PyNumber_Float(o);
  if (f == nullptr) throw PythonError();
  const double v = PyFloat_AS_DOUBLE(f);
  Py_DECREF(f);
  return v;
}

bool truth(PyObject *o) {
  const int v = PyObject_IsTrue(o);
  if (v < 0) throw PythonError();
  return v != 0;
}

void *pointer(const at::Tensor &t) { return t.data_ptr(); }

// Address of an optional tensor (None: null).
void *optional_pointer(PyObject *o, const char *what) { return o == Py_None ? nullptr : pointer(tensor(o, what)); }

// Extent and leading dimension of a row-major matrix on the device.
struct Dense {
  int64_t rows, cols, ld;
};
Dense dense2d(const at::Tensor &x, const char *what) {
  if (x.dim() != 2 || !x.is_cuda()) value_error(std::string(what) + " must be a 2-D device tensor");
  Dense d{x.size(0), x.size(1), 0};
  if (d.cols > 1 && x.stride(1) != 1) value_error(std::string(what) + " must be row-major (unit stride along columns)");
  d.ld = d.rows > 1 ? x.stride(0) : d.cols;
  if (d.ld < d.cols) value_error(std::string(what) + " has overlapping rows");
  return d;
}

// BSR_F32 / BSR_BF16, or BSR_ERR_DTYPE.
int dtype_code(const at::Tensor &t) {
  const auto s = t.scalar_type();
  return s == at::kFloat ? BSR_F32 : s == at::kBFloat16 ? BSR_BF16 : BSR_ERR_DTYPE;
}

// The stream's handle: `o` a torch stream or an integer, None for the current stream.
void *stream_handle(PyObject *o) {
  if (o == Py_None) return c10::hip::getCurrentHIPStream().stream();
  PyObject *h = PyObject_GetAttrString(o, "cuda_stream");
  if (h == nullptr) {
    PyErr_Clear();
    h = PyNumber_Long(o);
    if (h == nullptr) throw PythonError();
  }
  void *p = PyLong_AsVoidPtr(h);
  Py_DECREF(h);
  if (p == nullptr && PyErr_Occurred()) throw PythonError();
  return p;
}

at::Tensor new_tensor(at::IntArrayRef size, at::ScalarType type, const at::Tensor &like) {
  return at::empty(size, at::TensorOptions().dtype(type).device(like.device()));
}

// The workspace of a call: the caller's, or one of `need` bytes (none when need == 0).
struct Workspace {
  at::Tensor own;
  void *p = nullptr;
  size_t bytes = 0;
  Workspace(PyObject *given, size_t need, const at::Tensor &like) {
    if (given != Py_None) {
      const at::Tensor &t = tensor(given, "ws");
      p = pointer(t);
      bytes = (size_t)t.numel();
    } else if (need > 0) {
      own = new_tensor({(int64_t)need}, at::kByte, like);
      p = pointer(own);
      bytes = need;
    }
  }
};

// A tensor that the caller gave, or a new one: what goes back to Python, and its address.
struct Output {
  at::Tensor own;
  PyObject *given = Py_None;
  const at::Tensor &get() const { return given != Py_None ? THPVariable_Unpack(given) : own; }
  PyObject *result() const {
    if (given == Py_None) return THPVariable_Wrap(own);
    Py_INCREF(given);
    return given;
  }
};
Output output(PyObject *given, const char *what, at::IntArrayRef size, at::ScalarType type, const at::Tensor &like) {
  Output o;
  o.given = given;
  if (given == Py_None) o.own = new_tensor(size, type, like);
  else (void)tensor(given, what);
  return o;
}

int64_t blocks(int64_t n, int64_t b) { return b > 0 ? (n + b - 1) / b : 0; }

PyObject *code_result(int rc) { return PyLong_FromLong(rc); }

// Runs f, which calls the C library, without the GIL; it is held again however f ends.
struct GilReleased {
  PyThreadState *const save = PyEval_SaveThread();
  ~GilReleased() { PyEval_RestoreThread(save); }
};
template <typename F>
int released(F f) {
  const GilReleased guard;
  return f();
}

bool arity(Py_ssize_t n, Py_ssize_t want) {
  if (n == want) return true;
  PyErr_Format(PyExc_TypeError, "expected %zd arguments, got %zd", want, n);
  return false;
}

template <typename F>
PyObject *guarded(F f) {
  HANDLE_TH_ERRORS
  try {
    return f();
  } catch (const PythonError &) {
    return nullptr;
  }
  END_HANDLE_TH_ERRORS
}

// (X, br, bc, group_rows or None, keep, scores, want_scores, keep_mask, ws, stream) -> mask or (mask, scores)
PyObject *score_select(PyObject *, PyObject *const *a, Py_ssize_t n) {
  if (!arity(n, 10)) return nullptr;
  return guarded([&]() -> PyObject * {
    const at::Tensor &X = tensor(a[0], "X");
    const Dense x = dense2d(X, "X");
    const int br = extent(a[1]), bc = extent(a[2]);
    const int64_t nblocks = br > 0 && bc > 0 ? blocks(x.rows, br) * blocks(x.cols, bc) : 0;
    const bool with_scores = a[5] != Py_None || truth(a[6]);
    Output scores;
    if (with_scores) scores = output(a[5], "scores", {nblocks}, at::kDouble, X);
    const Output mask = output(a[7], "keep_mask", {nblocks}, at::kByte, X);
    const int code = dtype_code(X);
    if (code < 0) return code_result(code);
    const size_t need = a[8] == Py_None ? bsr_workspace_bytes(BSR_OP_SCORE_SELECT, x.rows, x.cols, 0, br, bc, code) : 0;
    const Workspace ws(a[8], need, X);
    const double keep = real(a[4]);
    const int64_t group_rows = a[3] == Py_None ? 0 : converted_integer(a[3]);
    void *stream = stream_handle(a[9]);
    void *px = pointer(X), *pm = pointer(mask.get());
    double *ps = with_scores ? static_cast<double *>(pointer(scores.get())) : nullptr;
    const bool grouped = a[3] != Py_None;
    const int rc = released([&] {
      return grouped ? bsr_score_select_grouped(px, code, x.rows, x.cols, x.ld, br, bc, group_rows, keep, ps,
                                                static_cast<uint8_t *>(pm), ws.p, ws.bytes, stream)
                     : bsr_score_select(px, code, x.rows, x.cols, x.ld, br, bc, keep, ps, static_cast<uint8_t *>(pm),
                                        ws.p, ws.bytes, stream);
    });
    if (rc != BSR_OK) return code_result(rc);
    if (!with_scores) return mask.result();
    return Py_BuildValue("(NN)", mask.result(), scores.result());
  });
}

// (X, br, bc, keep_mask, n_keep, row_ptr, col_idx, values, ws, stream) -> (row_ptr, col_idx, values)
PyObject *compress(PyObject *, PyObject *const *a, Py_ssize_t n) {
  if (!arity(n, 10)) return nullptr;
  return guarded([&]() -> PyObject * {
    const at::Tensor &X = tensor(a[0], "X");
    const Dense x = dense2d(X, "X");
    const int br = extent(a[1]), bc = extent(a[2]);
    // (a count that sizes an output has to be a whole number; one that does not is converted as by int())
    const int64_t n_keep = a[6] == Py_None || a[7] == Py_None ? integer(a[4]) : converted_integer(a[4]);
    const int64_t places = n_keep > 0 ? n_keep : 0;
    const Output row_ptr = output(a[5], "row_ptr", {blocks(x.rows, br) + 1}, at::kInt, X);
    const Output col_idx = output(a[6], "col_idx", {places}, at::kInt, X);
    const Output values = output(a[7], "values", {places, br, bc}, X.scalar_type(), X);
    const int code = dtype_code(X);
    if (code < 0) return code_result(code);
    const size_t need = a[8] == Py_None ? bsr_workspace_bytes(BSR_OP_COMPRESS, x.rows, x.cols, 0, br, bc, code) : 0;
    const Workspace ws(a[8], need, X);
    void *stream = stream_handle(a[9]);
    void *px = pointer(X), *pm = optional_pointer(a[3], "keep_mask"), *pv = pointer(values.get());
    int32_t *pr = static_cast<int32_t *>(pointer(row_ptr.get())), *pc = static_cast<int32_t *>(pointer(col_idx.get()));
    const int rc = released([&] {
      return bsr_compress(px, code, x.rows, x.cols, x.ld, br, bc, static_cast<const uint8_t *>(pm), n_keep, pr, pc, pv,
                          ws.p, ws.bytes, stream);
    });
    if (rc != BSR_OK) return code_result(rc);
    return Py_BuildValue("(NNN)", row_ptr.result(), col_idx.result(), values.result());
  });
}

// (row_ptr, col_idx, values, M, K, br, bc, out, stream) -> out
PyObject *decompress(PyObject *, PyObject *const *a, Py_ssize_t n) {
  if (!arity(n, 9)) return nullptr;
  return guarded([&]() -> PyObject * {
    const at::Tensor &values = tensor(a[2], "values");
    const int64_t M = integer(a[3]), K = integer(a[4]);
    const int br = extent(a[5]), bc = extent(a[6]);
    const Output out = output(a[7], "out", {M, K}, values.scalar_type(), values);
    const Dense o = dense2d(out.get(), "out");
    const int code = dtype_code(values);
    if (code < 0) return code_result(code);
    void *stream = stream_handle(a[8]);
    void *pr = optional_pointer(a[0], "row_ptr"), *pc = optional_pointer(a[1], "col_idx"), *pv = pointer(values);
    void *po = pointer(out.get());
    const int rc = released([&] {
      return bsr_decompress(static_cast<const int32_t *>(pr), static_cast<const int32_t *>(pc), pv, code, M, K, o.ld, br,
                            bc, po, stream);
    });
    return rc != BSR_OK ? code_result(rc) : out.result();
  });
}

// (row_ptr, col_idx, values, M, K, br, bc, dY, dW, accumulate, ws, stream) -> dW
PyObject *t_dense_matmul(PyObject *, PyObject *const *a, Py_ssize_t n) {
  if (!arity(n, 12)) return nullptr;
  return guarded([&]() -> PyObject * {
    const at::Tensor &dY = tensor(a[7], "dY"), &values = tensor(a[2], "values");
    const Dense y = dense2d(dY, "dY");
    const int64_t M = integer(a[3]), K = integer(a[4]);
    const int br = extent(a[5]), bc = extent(a[6]);
    if (y.rows != M) value_error("dY must have M rows");
    const bool accumulate = truth(a[9]);
    if (a[8] == Py_None && accumulate) value_error("accumulate needs an existing dW");
    const Output dW = output(a[8], "dW", {K, y.cols}, at::kFloat, dY);
    const Dense w = dense2d(dW.get(), "dW");
    const int code = dtype_code(dY);
    if (code < 0 || values.scalar_type() != dY.scalar_type()) return code_result(BSR_ERR_DTYPE);
    const size_t need =
        a[10] == Py_None ? bsr_workspace_bytes(BSR_OP_T_DENSE_MATMUL, M, K, y.cols, br, bc, code) : 0;
    const Workspace ws(a[10], need, dY);
    void *stream = stream_handle(a[11]);
    void *pr = optional_pointer(a[0], "row_ptr"), *pc = optional_pointer(a[1], "col_idx"), *pv = pointer(values);
    void *py = pointer(dY);
    float *pw = static_cast<float *>(pointer(dW.get()));
    const int rc = released([&] {
      return bsr_t_dense_matmul(static_cast<const int32_t *>(pr), static_cast<const int32_t *>(pc), pv, code, M, K, br,
                                bc, py, y.cols, y.ld, pw, w.ld, accumulate ? 1 : 0, ws.p, ws.bytes, stream);
    });
    return rc != BSR_OK ? code_result(rc) : dW.result();
  });
}

// (row_ptr, col_idx, values, M, K, br, bc, dY, dalpha, accumulate, ws, stream) -> dalpha
PyObject *affine_scale_grad(PyObject *, PyObject *const *a, Py_ssize_t n) {
  if (!arity(n, 12)) return nullptr;
  return guarded([&]() -> PyObject * {
    const at::Tensor &dY = tensor(a[7], "dY"), &values = tensor(a[2], "values");
    const Dense y = dense2d(dY, "dY");
    const int64_t M = integer(a[3]), K = integer(a[4]);
    const int br = extent(a[5]), bc = extent(a[6]);
    if (y.rows != M || y.cols != K) value_error("dY must be [M x K]");
    const bool accumulate = truth(a[9]);
    if (a[8] == Py_None && accumulate) value_error("accumulate needs an existing dalpha");
    const Output dalpha = output(a[8], "dalpha", {K}, at::kFloat, dY);
    const int code = dtype_code(dY);
    if (code < 0 || values.scalar_type() != dY.scalar_type()) return code_result(BSR_ERR_DTYPE);
    const size_t need = a[10] == Py_None ? bsr_workspace_bytes(BSR_OP_AFFINE_SCALE_GRAD, M, K, 0, br, bc, code) : 0;
    const Workspace ws(a[10], need, dY);
    void *stream = stream_handle(a[11]);
    void *pr = optional_pointer(a[0], "row_ptr"), *pc = optional_pointer(a[1], "col_idx"), *pv = pointer(values);
    void *py = pointer(dY);
    float *pa = static_cast<float *>(pointer(dalpha.get()));
    const int rc = released([&] {
      return bsr_affine_scale_grad(static_cast<const int32_t *>(pr), static_cast<const int32_t *>(pc), pv, code, M, K, br,
                                   bc, py, y.ld, pa, accumulate ? 1 : 0, ws.p, ws.bytes, stream);
    });
    return rc != BSR_OK ? code_result(rc) : dalpha.result();
  });
}

// () -> handle of the current stream of the current device
PyObject *current_stream(PyObject *, PyObject *) {
  return guarded([&]() -> PyObject * { return PyLong_FromVoidPtr(c10::hip::getCurrentHIPStream().stream()); });
}

PyMethodDef methods[] = {
    {"score_select", reinterpret_cast<PyCFunction>(reinterpret_cast<void *>(score_select)), METH_FASTCALL, nullptr},
    {"compress", reinterpret_cast<PyCFunction>(reinterpret_cast<void *>(compress)), METH_FASTCALL, nullptr},
    {"decompress", reinterpret_cast<PyCFunction>(reinterpret_cast<void *>(decompress)), METH_FASTCALL, nullptr},
    {"t_dense_matmul", reinterpret_cast<PyCFunction>(reinterpret_cast<void *>(t_dense_matmul)), METH_FASTCALL, nullptr},
    {"affine_scale_grad", reinterpret_cast<PyCFunction>(reinterpret_cast<void *>(affine_scale_grad)), METH_FASTCALL, nullptr},
    {"current_stream", current_stream, METH_NOARGS, nullptr},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_torch_calls", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

extern "C" PyObject *PyInit__torch_calls() { return PyModule_Create(&module); }
