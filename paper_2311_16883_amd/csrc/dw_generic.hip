// Weight gradient from a BSR activation, any block shape (paper Sec. III, Fig. 2:
// dW = Xhat^T * dY, "BSpMM").  Plain binary32 FMA path: used for block shapes
// and element types the matrix-core kernel does not cover.
//
// A workgroup owns a 64 x 64 tile of dW and a contiguous range of block-rows
// (split of the contraction).  Per block-row it looks up which block-columns of
// its tile are kept (LDS table), stages 16 rows of the kept blocks (zeros where
// pruned) and of dY in LDS and accumulates 4 x 4 outputs per thread.  Block-rows
// without a kept block in the tile are skipped.  With more than one split the
// partial tiles go to the workspace and are summed in a fixed order afterwards.
#include "common.h"

namespace bsr {

namespace {

constexpr int TK = 64, TN = 64, RM = 16;

template <typename T>
__global__ __launch_bounds__(256) void dw_generic_kernel(
    const int32_t *__restrict__ row_ptr, const int32_t *__restrict__ col_idx,
    const T *__restrict__ values, int64_t M, int64_t K, int br, int bc, int64_t nbr, int64_t nbc,
    const T *__restrict__ dY, int64_t N, int64_t lddy, float *__restrict__ out, int64_t ldo,
    int64_t split_stride, int64_t rows_per_split, int accumulate) {
  __shared__ float A[RM][TK];
  __shared__ float B[RM][TN];
  __shared__ int32_t slot[TK];

  const int t = threadIdx.x, tx = t & 15, ty = t >> 4;
  const int64_t k0 = (int64_t)blockIdx.x * TK, n0 = (int64_t)blockIdx.y * TN;
  const int64_t i_begin = (int64_t)blockIdx.z * rows_per_split;
  const int64_t i_end = (i_begin + rows_per_split) < nbr ? (i_begin + rows_per_split) : nbr;
  const int64_t jfirst = k0 / bc;
  int64_t jlast = (k0 + TK - 1) / bc;
  if (jlast > nbc - 1) jlast = nbc - 1;
  const int ncol = (int)(jlast - jfirst + 1);

  float acc[4][4];
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b) acc[a][b] = 0.f;

  for (int64_t i = i_begin; i < i_end; ++i) {
    if (t < ncol) slot[t] = -1;
    __syncthreads();
    const int64_t p0 = row_ptr[i], p1 = row_ptr[i + 1];
    int hit = 0;
    for (int64_t p = p0 + t; p < p1; p += 256) {
      const int64_t j = col_idx[p];
      if (j >= jfirst && j <= jlast) {
        slot[j - jfirst] = (int32_t)p;
        hit = 1;
      }
    }
    if (!__syncthreads_or(hit)) continue;

    for (int r0 = 0; r0 < br; r0 += RM) {
      for (int e = t; e < RM * TK; e += 256) {
        const int rr = e / TK, kk = e % TK;
        const int64_t k = k0 + kk;
        const int r = r0 + rr;
        float v = 0.f;
        if (k < K && r < br) {
          const int64_t j = k / bc;
          const int32_t p = slot[j - jfirst];
          if (p >= 0) v = elem_to_float<T>(values[((int64_t)p * br + r) * bc + (k - j * bc)]);
        }
        A[rr][kk] = v;
      }
      for (int e = t; e < RM * TN; e += 256) {
        const int rr = e / TN, nn = e % TN;
        const int64_t m = i * br + r0 + rr, n = n0 + nn;
        float v = 0.f;
        if (r0 + rr < br && m < M && n < N) v = elem_to_float<T>(dY[m * lddy + n]);
        B[rr][nn] = v;
      }
      __syncthreads();
#pragma unroll
      for (int rr = 0; rr < RM; ++rr) {
        float a[4], b[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          a[u] = A[rr][ty * 4 + u];
          b[u] = B[rr][tx * 4 + u];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
          for (int w = 0; w < 4; ++w) acc[u][w] = fmaf(a[u], b[w], acc[u][w]);
      }
      __syncthreads();
    }
  }

  float *o = out + (int64_t)blockIdx.z * split_stride;
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int64_t k = k0 + ty * 4 + u;
    if (k >= K) continue;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const int64_t n = n0 + tx * 4 + w;
      if (n >= N) continue;
      float *dst = o + k * ldo + n;
      *dst = accumulate ? *dst + acc[u][w] : acc[u][w];
    }
  }
}

__global__ __launch_bounds__(256) void splitk_reduce_kernel(const float *__restrict__ partial,
                                                            int splits, int64_t K, int64_t N,
                                                            float *__restrict__ dW, int64_t lddw,
                                                            int accumulate) {
  const int64_t total = K * N;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t k = e / N, n = e % N;
    float s = accumulate ? dW[k * lddw + n] : 0.f;
    for (int sp = 0; sp < splits; ++sp) s += partial[(int64_t)sp * total + e];
    dW[k * lddw + n] = s;
  }
}

// Same sum, four columns per thread (N, lddw and the pointers allow 16-byte access).
__global__ __launch_bounds__(256) void splitk_reduce4_kernel(const float4 *__restrict__ partial,
                                                             int splits, int64_t K, int64_t N4,
                                                             float *__restrict__ dW, int64_t lddw,
                                                             int accumulate) {
  const int64_t total4 = K * N4;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total4;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t k = e / N4, n4 = e % N4;
    float4 *dst = reinterpret_cast<float4 *>(dW + k * lddw) + n4;
    float4 s = accumulate ? *dst : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 4
    for (int sp = 0; sp < splits; ++sp) {
      const float4 v = partial[(int64_t)sp * total4 + e];
      s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
    }
    *dst = s;
  }
}

// ... and for many splits of a small dW, where the kernels above are a few workgroups with a long chain of loads each: a
// thread has eight partial matrices' loads on their way, and `groups` threads share an output vector, each with a part of
// the splits; their sums meet in LDS.  Always the same order: splits ascending inside a part, then the parts.  V = float4 (as
// above) or float.  (Partial matrices of [196 x 196], 64 splits: 7.5 -> 4.0 us; whole dW calls [26212 x 141 x 130] 27.1 -> 16.7,
// [13620 x 96 x 32] 14.6 -> 11.4.  Of few splits the simpler kernels are faster: [3000 x 400 x 300], nine splits, 13.7 and 14.8.)
constexpr int kReduceInFlight = 8;
__device__ __forceinline__ float4 add(const float4 &a, const float4 &b) {
  return make_float4(a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w);
}
__device__ __forceinline__ float add(float a, float b) { return a + b; }

struct SharedReduceBatch {
  ReduceJob it[kReduceBatchMax];
  uint32_t wg_begin[kReduceBatchMax + 1];
  uint8_t groups[kReduceBatchMax];
};

inline __host__ __device__ bool reduce_by_vectors(const ReduceJob &j) {
  return j.N % 4 == 0 && j.lddw % 4 == 0 && (uintptr_t)j.dW % 16 == 0 && (uintptr_t)j.partial % 16 == 0;
}

inline int64_t reduce_outputs(const ReduceJob &j) { return reduce_by_vectors(j) ? j.K * j.N / 4 : j.K * j.N; }

// Threads that share an output of a product, 1: the simpler kernels do.  (`outs` = outputs of all products of the launch: as
// many threads as the chip has room for, each with four splits or more.  Beyond kReduceSharedVectors the simpler kernels have
// enough of them for vectors: whole dW calls of M = 50176 with them and so, [300 x 300] 37.4 and 35.9 us, [1000 x 128] 1.3 %
// less, [512 x 512] and [768 x 384] 2 % more; entry by entry, [300 x 301], 38.9 and 30.9.)
constexpr int64_t kReduceSharedVectors = 128 * 256;
int reduce_groups(const ReduceJob &j, int64_t outs) {
  if (j.splits < 16 || (reduce_by_vectors(j) && outs > kReduceSharedVectors)) return 1;
  int groups = 1;
  while (groups < 16 && outs * groups < 512 * 256 && j.splits >= 8 * groups) groups *= 2;
  return groups;
}

template <typename V>
__device__ __forceinline__ void shared_reduce_body(const ReduceJob &it, const uint32_t groups, const uint32_t wg,
                                                   const uint32_t wgs, V *sh) {
  const int64_t nv = it.N / (int64_t)(sizeof(V) / 4), total = it.K * nv;
  const V *partial = reinterpret_cast<const V *>(it.partial);
  const uint32_t per = 256u / groups, t = threadIdx.x, o = t % per, g = t / per;
  const int lo = (int)((uint32_t)it.splits * g / groups), hi = (int)((uint32_t)it.splits * (g + 1) / groups);
  for (int64_t base = (int64_t)wg * per; base < total; base += (int64_t)wgs * per) {
    const int64_t e = base + o;
    const V *src = partial + (e < total ? e : total - 1);
    V s{};
    for (int sp = lo; sp < hi; sp += kReduceInFlight) {
      V v[kReduceInFlight];
#pragma unroll
      for (int k = 0; k < kReduceInFlight; ++k) v[k] = src[(int64_t)(sp + k < hi ? sp + k : hi - 1) * total];
#pragma unroll
      for (int k = 0; k < kReduceInFlight; ++k)
        if (sp + k < hi) s = add(s, v[k]);
    }
    sh[t] = s;
    __syncthreads();
    if (g == 0 && e < total) {
      for (uint32_t q = 1; q < groups; ++q) s = add(s, sh[q * per + o]);
      const int64_t k = e / nv;
      V *dst = reinterpret_cast<V *>(it.dW + k * it.lddw) + (e - k * nv);
      *dst = it.accumulate ? add(*dst, s) : s;
    }
    __syncthreads();
  }
}

template <typename V>
__global__ __launch_bounds__(256) void splitk_reduce_shared_kernel(ReduceJob job, uint32_t groups) {
  __shared__ V sh[256];
  shared_reduce_body<V>(job, groups, blockIdx.x, gridDim.x, sh);
}

__global__ __launch_bounds__(256) void splitk_reduce_shared_batched_kernel(SharedReduceBatch b, int n) {
  __shared__ float4 sh[256];
  int i = 0;
  while (i + 1 < n && blockIdx.x >= b.wg_begin[i + 1]) ++i;
  const ReduceJob &it = b.it[i];
  const uint32_t wg = blockIdx.x - b.wg_begin[i], wgs = b.wg_begin[i + 1] - b.wg_begin[i];
  if (reduce_by_vectors(it)) shared_reduce_body<float4>(it, b.groups[i], wg, wgs, sh);
  else shared_reduce_body<float>(it, b.groups[i], wg, wgs, reinterpret_cast<float *>(sh));
}

inline int64_t shared_reduce_wgs(const ReduceJob &j, int groups) {
  return ceil_div(reduce_outputs(j) * groups, (int64_t)256);
}

// The same sums for several tensors in one launch (item = tensor, found from the prefix of
// workgroup counts); per element the order of the additions is that of the kernels above.
struct ReduceBatch {
  ReduceJob it[kReduceBatchMax];
  uint32_t wg_begin[kReduceBatchMax + 1];
};

__global__ __launch_bounds__(256) void splitk_reduce_batched_kernel(ReduceBatch b, int n) {
  int i = 0;
  while (i + 1 < n && blockIdx.x >= b.wg_begin[i + 1]) ++i;
  const ReduceJob &it = b.it[i];
  const int64_t wg = blockIdx.x - b.wg_begin[i], wgs = b.wg_begin[i + 1] - b.wg_begin[i];
  const bool vec = it.N % 4 == 0 && it.lddw % 4 == 0 && (uintptr_t)it.dW % 16 == 0 && (uintptr_t)it.partial % 16 == 0;
  if (vec) {
    const int64_t N4 = it.N / 4, total4 = it.K * N4;
    const float4 *partial = reinterpret_cast<const float4 *>(it.partial);
    for (int64_t e = wg * 256 + threadIdx.x; e < total4; e += wgs * 256) {
      const int64_t k = e / N4, n4 = e % N4;
      float4 *dst = reinterpret_cast<float4 *>(it.dW + k * it.lddw) + n4;
      float4 s = it.accumulate ? *dst : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 4
      for (int sp = 0; sp < it.splits; ++sp) {
        const float4 v = partial[(int64_t)sp * total4 + e];
        s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
      }
      *dst = s;
    }
  } else {
    const int64_t total = it.K * it.N;
    for (int64_t e = wg * 256 + threadIdx.x; e < total; e += wgs * 256) {
      const int64_t k = e / it.N, c = e % it.N;
      float s = it.accumulate ? it.dW[k * it.lddw + c] : 0.f;
      for (int sp = 0; sp < it.splits; ++sp) s += it.partial[(int64_t)sp * total + e];
      it.dW[k * it.lddw + c] = s;
    }
  }
}

int generic_splits(int64_t M, int64_t K, int64_t N, int br) {
  const int64_t nbr = ceil_div(M, br);
  const int64_t tiles = ceil_div(K, TK) * ceil_div(N, TN);
  int64_t s = 2048 / (tiles > 0 ? tiles : 1);
  if (s < 1) s = 1;
  if (s > nbr) s = nbr;
  if (s > 64) s = 64;
  if (s < 1) s = 1;
  return (int)s;
}

}  // namespace

int launch_splitk_reduce(const float *partial, int splits, int64_t K, int64_t N, float *dW,
                         int64_t lddw, int accumulate, hipStream_t s) {
  const int64_t total = K * N;
  if (total == 0) return BSR_OK;
  const ReduceJob job{partial, dW, K, N, lddw, splits, accumulate};
  const int groups = reduce_groups(job, reduce_outputs(job));
  const bool vec = reduce_by_vectors(job);
  if (groups > 1) {
    const dim3 grid((unsigned)shared_reduce_wgs(job, groups));
    if (vec) hipLaunchKernelGGL((splitk_reduce_shared_kernel<float4>), grid, dim3(256), 0, s, job, (uint32_t)groups);
    else hipLaunchKernelGGL((splitk_reduce_shared_kernel<float>), grid, dim3(256), 0, s, job, (uint32_t)groups);
    return check_launch();
  }
  if (vec) {
    const int64_t blocks = ceil_div(total / 4, 256);
    hipLaunchKernelGGL(splitk_reduce4_kernel, dim3((unsigned)(blocks < 8192 ? blocks : 8192)),
                       dim3(256), 0, s, reinterpret_cast<const float4 *>(partial), splits, K, N / 4,
                       dW, lddw, accumulate);
    return check_launch();
  }
  const int64_t blocks = ceil_div(total, 256);
  hipLaunchKernelGGL(splitk_reduce_kernel, dim3((unsigned)(blocks < 8192 ? blocks : 8192)), dim3(256),
                     0, s, partial, splits, K, N, dW, lddw, accumulate);
  return check_launch();
}

int launch_splitk_reduce_batched(const ReduceJob *jobs, int n, hipStream_t s) {
  for (int i0 = 0; i0 < n; i0 += kReduceBatchMax) {
    const int m = n - i0 < kReduceBatchMax ? n - i0 : kReduceBatchMax;
    const ReduceJob *const job = jobs + i0;
    int64_t outs = 0;
    for (int i = 0; i < m; ++i) outs += reduce_outputs(job[i]);
    bool shared = false;
    for (int i = 0; i < m; ++i) shared = shared || reduce_groups(job[i], outs) > 1;
    uint32_t wgs = 0;
    if (shared) {                     // (one launch for all: a second one costs more than the other kernel saves the rest)
      SharedReduceBatch c;
      for (int i = 0; i < m; ++i) {
        const int groups = reduce_groups(job[i], outs);
        c.it[i] = job[i];
        c.groups[i] = (uint8_t)groups;
        c.wg_begin[i] = wgs;
        wgs += (uint32_t)shared_reduce_wgs(job[i], groups);
      }
      c.wg_begin[m] = wgs;
      hipLaunchKernelGGL(splitk_reduce_shared_batched_kernel, dim3(wgs), dim3(256), 0, s, c, m);
    } else {
      ReduceBatch b;
      for (int i = 0; i < m; ++i) {
        b.it[i] = job[i];
        b.wg_begin[i] = wgs;
        const int64_t blocks = ceil_div(ceil_div(job[i].K * job[i].N, 4), 256);
        wgs += (uint32_t)(blocks < 1 ? 1 : (blocks < 2048 ? blocks : 2048));
      }
      b.wg_begin[m] = wgs;
      hipLaunchKernelGGL(splitk_reduce_batched_kernel, dim3(wgs), dim3(256), 0, s, b, m);
    }
    const int rc = check_launch();
    if (rc != BSR_OK) return rc;
  }
  return BSR_OK;
}

size_t dw_generic_ws_bytes(int64_t M, int64_t K, int64_t N, int br, int bc) {
  (void)bc;
  const int s = generic_splits(M, K, N, br);
  return s > 1 ? (size_t)s * (size_t)K * (size_t)N * sizeof(float) : 0;
}

int launch_dw_generic(const int32_t *row_ptr, const int32_t *col_idx, const void *values, int dtype,
                      int64_t M, int64_t K, int br, int bc, const void *dY, int64_t N, int64_t lddy,
                      float *dW, int64_t lddw, int accumulate, void *ws, size_t ws_bytes,
                      hipStream_t s) {
  if (K == 0 || N == 0) return BSR_OK;
  const int64_t nbr = ceil_div(M, br), nbc = ceil_div(K, bc);
  const int splits = generic_splits(M, K, N, br);
  if (splits > 1 && (ws == nullptr || ws_bytes < dw_generic_ws_bytes(M, K, N, br, bc)))
    return BSR_ERR_WORKSPACE;
  const int64_t rps = nbr > 0 ? ceil_div(nbr, splits) : 1;
  float *out = splits > 1 ? static_cast<float *>(ws) : dW;
  const int64_t ldo = splits > 1 ? N : lddw;
  const int64_t stride = splits > 1 ? K * N : 0;
  const int acc_direct = splits > 1 ? 0 : accumulate;
  dim3 grid((unsigned)ceil_div(K, TK), (unsigned)ceil_div(N, TN), (unsigned)splits);
  if (dtype == BSR_F32)
    hipLaunchKernelGGL((dw_generic_kernel<float>), grid, dim3(256), 0, s, row_ptr, col_idx,
                       static_cast<const float *>(values), M, K, br, bc, nbr, nbc,
                       static_cast<const float *>(dY), N, lddy, out, ldo, stride, rps, acc_direct);
  else
    hipLaunchKernelGGL((dw_generic_kernel<uint16_t>), grid, dim3(256), 0, s, row_ptr, col_idx,
                       static_cast<const uint16_t *>(values), M, K, br, bc, nbr, nbc,
                       static_cast<const uint16_t *>(dY), N, lddy, out, ldo, stride, rps, acc_direct);
  int rc = check_launch();
  if (rc != BSR_OK || splits == 1) return rc;
  return launch_splitk_reduce(out, splits, K, N, dW, lddw, accumulate, s);
}

}  // namespace bsr
