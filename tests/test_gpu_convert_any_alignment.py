"""Mask -> BSR of matrices whose rows or block widths are no whole 16-byte vectors."""
import numpy as np
import pytest
import torch

import oracle
from paper_2311_16883_amd import binding as B
from test_dw_dispatch import recorder  # noqa: F401
from test_gpu_parity import rand_pair, to_dev, to_host

ANY_ALIGNMENT = [
    (1400, 1301, 14, 14, 0, 0.5),      # rows on odd elements, blocks of a vector and three quarters, a column of one in the last
    (1393, 1302, 14, 14, 5, 0.9),      # a last block-row of seven rows, far rows
    (200, 4000, 9, 13, 1, 0.3),
    (61, 9, 14, 9, 0, 1.0),            # one vector and one element; a row is little more
    (2000, 9, 300, 9, 1, 1.0),         # ... in blocks that have enough of them
    (700, 1002, 12, 30, 2, 0.5),       # pieces of 8 bytes or 4 in binary32
    (30000, 71, 1, 32, 0, 0.4),        # many block-rows: a wave for each
    (30003, 131, 1, 9, 3, 0.6),
    (40001, 201, 2, 14, 0, 0.02),      # block-rows that keep nothing
    (9000, 2301, 1, 32, 0, 1.0),       # 72 block-columns, two passes of a wave
    (30000, 71, 1, 32, 1, 0.4),        # (rows apart: binary32 as well)
    (9000, 2301, 1, 32, 2, 1.0),
    (9000, 61, 1, 128, 1, 0.5),        # many block-rows of one block: a workgroup each
]


def test_conversions_by_kernel(recorder):  # noqa: F811
    """Vectors that end with the row, and a wave for a block-row, where there is enough for them; the list below takes both."""
    def names(dtype, shapes):
        got = recorder([dict(compress=dict(M=M, K=K, br=br, bc=bc, ldx=K + pad), dtype=dtype) for M, K, br, bc, pad, *_ in shapes])
        assert [g["rc"] for g in got] == [0] * len(got)
        return ["tail" if "compress_kernelILi3E" in g["names"][-1] else "rows" if "compress_rows" in g["names"][-1] else "other" for g in got]

    for dtype in (0, 1):
        assert names(dtype, [(49000, 30, 1, 64, 1), (49000, 60, 1, 128, 1), (20000, 322, 3, 17, 1), (41000, 161, 7, 9, 1)]) == ["other"] * 4
        assert names(dtype, [(41298, 805, 14, 14, 0), (9170, 1779, 14, 14, 0), (5000, 805, 7, 9, 0)]) == ["tail"] * 3
        assert names(dtype, [(10307, 1071, 1, 32, 1), (30000, 601, 1, 32, 1), (41000, 805, 7, 9, 0)]) == ["rows"] * 3
        span = [] if dtype else [6, 8, 9]     # (contiguous rows of whole words)
        reached = ["tail"] * 3 + ["other"] + ["tail"] * 2 + ["rows"] * 6 + ["other"]
        assert names(dtype, ANY_ALIGNMENT) == ["other" if i in span else n for i, n in enumerate(reached)]
    assert names(0, [(29297, 1618, 9, 13, 0), (20466, 2669, 14, 14, 0)]) == ["other"] * 2
    assert names(1, [(29297, 1618, 9, 13, 0), (20466, 2669, 14, 14, 0)]) == ["tail"] * 2


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("M,K,br,bc,pad,keep", ANY_ALIGNMENT)
def test_mask_to_bsr_at_any_alignment(M, K, br, bc, pad, keep, dtype):
    """Bit for bit what the oracle stores; alone and in a batch, from a buffer that ends with the last element and from the
    middle of NaN (between the rows, too); nothing is written behind the results."""
    X, _ = rand_pair(M, K, 8, dtype, seed=M + K)
    _, o_mask, o_rp, o_ci, o_val = oracle.prune(X, br, bc, keep)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    flat = torch.full((M * (K + pad) + 64,), float("nan"), device="cuda", dtype=dt)
    inner = flat[33:].as_strided((M, K), (K + pad, 1))
    inner.copy_(to_dev(X))
    last = flat[:(M - 1) * (K + pad) + K].clone().as_strided((M, K), (K + pad, 1))
    last.copy_(inner)
    mask, n = torch.from_numpy(o_mask.reshape(-1).astype(np.uint8)).cuda(), len(o_ci)
    outs = []
    for x in (inner, last):
        values = torch.full((n * br * bc + 64,), 7.0, device="cuda", dtype=dt)
        out = (torch.empty(len(o_rp), dtype=torch.int32, device="cuda"), torch.empty(n, dtype=torch.int32, device="cuda"),
               values[:n * br * bc].view(n, br, bc))
        B.bsr_compress_batched(B.CompressBatch([(x, br, bc, mask, n, *out)]))
        outs += [out, B.bsr_compress(x, br, bc, mask, n)]
        assert (values[n * br * bc:] == 7.0).all()
    torch.cuda.synchronize()
    for rp, ci, val in outs:
        assert np.array_equal(rp.cpu().numpy(), o_rp) and np.array_equal(ci.cpu().numpy(), o_ci)
        assert to_host(val).tobytes() == o_val.tobytes()
