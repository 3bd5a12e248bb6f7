"""Runs calls of the library against tests/launch_recorder.c and prints what they would launch (a program of its own: it must
not share a process with torch, which loads the real runtime).

argv: the recorder, the library.  stdin: a JSON list of calls; stdout: a JSON list of
{"rc", "ws", "kernels": [[kernel, workgroups], ...]}, ws = what the workspace query returns.
A call: {"items": [{M, K, N, b or br + bc, lddy, lddw, dY, values, accumulate}, ...], "dtype", "batched"} for weight gradients, or
{"select": {M, K, br, bc, ldx, X}, "dtype"} for bsr_score_select, or {"compress": the same, "dtype"} for bsr_compress; addresses are numbers that nothing reads.  The workspace passed
is exactly the one the query asks for.
"""
import ctypes as C
import json
import sys

ADDRESS = 1 << 20


class MatmulItem(C.Structure):
    _fields_ = [("row_ptr", C.c_void_p), ("col_idx", C.c_void_p), ("values", C.c_void_p), ("M", C.c_int64),
                ("K", C.c_int64), ("br", C.c_int32), ("bc", C.c_int32), ("dY", C.c_void_p), ("N", C.c_int64),
                ("lddy", C.c_int64), ("dW", C.c_void_p), ("lddw", C.c_int64), ("accumulate", C.c_int32)]


def main():
    recorder = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
    lib = C.CDLL(sys.argv[2])
    recorder.recorder_name.restype = C.c_char_p
    recorder.recorder_workgroups.restype = C.c_uint64
    i64, i32, p, size = C.c_int64, C.c_int, C.c_void_p, C.c_size_t
    lib.bsr_workspace_bytes.restype = size
    lib.bsr_workspace_bytes.argtypes = [i32, i64, i64, i64, i32, i32, i32]
    lib.bsr_t_dense_matmul.argtypes = [p, p, p, i32, i64, i64, i32, i32, p, i64, i64, p, i64, i32, p, size, p]
    lib.bsr_t_dense_matmul_batched_workspace_bytes.restype = size
    lib.bsr_t_dense_matmul_batched_workspace_bytes.argtypes = [p, i32, i32]
    lib.bsr_t_dense_matmul_batched.argtypes = [p, i32, i32, p, size, p]
    lib.bsr_score_select.argtypes = [p, i32, i64, i64, i64, i32, i32, C.c_double, p, p, p, size, p]
    lib.bsr_compress.argtypes = [p, i32, i64, i64, i64, i32, i32, p, i64, p, p, p, p, size, p]
    out = []

    def launched():
        return [[recorder.recorder_name(i).decode(), recorder.recorder_workgroups(i)] for i in range(recorder.recorder_count())]

    for call in json.load(sys.stdin):
        if "select" in call or "compress" in call:
            a, dtype = call.get("select") or call["compress"], call.get("dtype", 1)
            M, K, br, bc = a["M"], a["K"], a["br"], a["bc"]
            recorder.recorder_reset()
            if "compress" in call:
                ws = lib.bsr_workspace_bytes(1, M, K, 0, br, bc, dtype)
                rc = lib.bsr_compress(a.get("X", ADDRESS), dtype, M, K, a.get("ldx", K), br, bc, ADDRESS, -(-M // br), ADDRESS, ADDRESS,
                                      ADDRESS, ADDRESS, ws, None)
                out.append({"rc": rc, "ws": ws, "kernels": launched()})
                continue
            ws = lib.bsr_workspace_bytes(0, M, K, 0, br, bc, dtype)
            rc = lib.bsr_score_select(a.get("X", ADDRESS), dtype, M, K, a.get("ldx", K), br, bc, 0.5, None, ADDRESS, ADDRESS, ws, None)
            out.append({"rc": rc, "ws": ws, "kernels": launched()})
            continue
        dtype, items = call.get("dtype", 1), (MatmulItem * len(call["items"]))()
        for a, it in zip(items, call["items"]):
            a.row_ptr = a.col_idx = a.dW = ADDRESS
            a.values, a.dY = it.get("values", ADDRESS), it.get("dY", ADDRESS)
            a.M, a.K, a.N = it["M"], it["K"], it["N"]
            a.br, a.bc = it.get("br", it.get("b")), it.get("bc", it.get("b"))
            a.lddy, a.lddw, a.accumulate = it.get("lddy", a.N), it.get("lddw", a.N), it.get("accumulate", 0)
        recorder.recorder_reset()
        if call.get("batched", len(items) > 1):
            ws = lib.bsr_t_dense_matmul_batched_workspace_bytes(items, len(items), dtype)
            rc = lib.bsr_t_dense_matmul_batched(items, len(items), dtype, ADDRESS, ws, None)
        else:
            a = items[0]
            ws = lib.bsr_workspace_bytes(3, a.M, a.K, a.N, a.br, a.bc, dtype)
            rc = lib.bsr_t_dense_matmul(a.row_ptr, a.col_idx, a.values, dtype, a.M, a.K, a.br, a.bc, a.dY, a.N, a.lddy, a.dW,
                                        a.lddw, a.accumulate, ADDRESS, ws, None)
        out.append({"rc": rc, "ws": ws, "kernels": launched()})
    json.dump(out, sys.stdout)


if __name__ == "__main__":
    main()
