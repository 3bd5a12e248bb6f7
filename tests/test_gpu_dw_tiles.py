"""dW of products on their own that the 128x128 tiles take, as they are or re-tiled from other block shapes: which forms of the
kernel the sizes below reach (CPU), and their results."""
import re

import numpy as np
import pytest
import torch

import oracle
from paper_2311_16883_amd import binding as B
from test_dw_dispatch import recorder  # noqa: F401
from test_gpu_parity import DW_TOL, DW_TOL_DERIVED, dw_error, rand_pair, to_dev

# Type, block, form of the kernel (rows of dY on odd elements; binary32 14x14 blocks in slots or packed), splits; M, K, N.  Ragged
# rows and columns, few rows and many, wide and narrow.
TILES = [
    ("f32", 14, 14, "plain", False, 27, 3928, 9), ("f32", 14, 14, "plain", True, 957, 41, 14),
    ("f32", 14, 14, "packed", False, 24, 2862, 1160), ("f32", 14, 14, "packed", True, 1961, 3817, 8),
    ("f32", 16, 16, "plain", False, 21, 1541, 1242), ("f32", 16, 16, "plain", True, 2174, 2086, 40),
    ("f32", 32, 32, "plain", False, 34, 2831, 294), ("f32", 32, 32, "plain", True, 794, 46, 14),
    ("f32", 64, 64, "plain", False, 21, 2690, 404), ("f32", 64, 64, "plain", True, 898, 86, 12),
    ("bf16", 14, 14, "plain", False, 31, 3063, 258), ("bf16", 14, 14, "plain", True, 2889, 54, 20),
    ("bf16", 14, 14, "odd", False, 51, 1470, 271), ("bf16", 14, 14, "odd", True, 1994, 49, 13),
    ("bf16", 16, 16, "plain", False, 22, 2088, 724), ("bf16", 16, 16, "plain", True, 2543, 54, 8),
    ("bf16", 16, 16, "odd", False, 25, 3379, 265), ("bf16", 16, 16, "odd", True, 3062, 95, 13),
    ("bf16", 32, 32, "plain", False, 40, 3233, 152), ("bf16", 32, 32, "plain", True, 2455, 75, 8),
    ("bf16", 32, 32, "odd", False, 46, 2429, 97), ("bf16", 32, 32, "odd", True, 2455, 46, 15),
    ("bf16", 64, 64, "plain", False, 34, 2764, 138), ("bf16", 64, 64, "plain", True, 2314, 56, 8),
    ("bf16", 64, 64, "odd", False, 36, 3614, 73), ("bf16", 64, 64, "odd", True, 2427, 57, 9),
]

# ... in block shapes that are re-tiled first.
RETILED = [
    ("f32", 1, 32, "plain", False, 125, 3450, 22), ("f32", 1, 32, "plain", True, 671, 55, 8),
    ("f32", 1, 8, "plain", False, 189, 425, 20), ("f32", 1, 8, "plain", True, 660, 44, 10),
    ("f32", 1, 96, "plain", False, 20, 1843, 1246), ("f32", 1, 96, "plain", True, 459, 41, 8),
    ("f32", 8, 16, "plain", False, 123, 3827, 37), ("f32", 8, 16, "plain", True, 1906, 57, 10),
    ("bf16", 1, 32, "plain", False, 195, 2197, 10), ("bf16", 1, 32, "plain", True, 1867, 59, 10),
    ("bf16", 1, 32, "odd", False, 278, 1836, 9), ("bf16", 1, 32, "odd", True, 1794, 60, 11),
    ("bf16", 1, 8, "plain", False, 255, 72, 14), ("bf16", 1, 8, "plain", True, 515, 41, 14),
    ("bf16", 1, 8, "odd", False, 407, 77, 11), ("bf16", 1, 8, "odd", True, 933, 43, 23),
    ("bf16", 1, 96, "plain", False, 26, 3293, 580), ("bf16", 1, 96, "plain", True, 1756, 41, 22),
    ("bf16", 1, 96, "odd", False, 27, 3404, 939), ("bf16", 1, 96, "odd", True, 2454, 56, 11),
    ("bf16", 8, 16, "plain", False, 492, 880, 36), ("bf16", 8, 16, "plain", True, 2928, 44, 14),
    ("bf16", 8, 16, "odd", False, 313, 1214, 41), ("bf16", 8, 16, "odd", True, 2083, 50, 35),
]


def placements(form):
    """(elements that a row of dY has beyond N, elements in front of it), such that the form is the same."""
    return ((0, 0), (1, 0), (2, 1)) if form == "odd" else ((0, 0), (2, 2))


@pytest.mark.parametrize("cases", [TILES, RETILED])
def test_the_sizes_below_reach_the_tiles(recorder, cases):  # noqa: F811
    for dtype, br, bc, form, splits, M, K, N in cases:
        size = 4 if dtype == "f32" else 2
        got = recorder([dict(items=[dict(M=M, K=K, N=N, br=br, bc=bc, lddy=N + pad, dY=(1 << 20) + shift * size)],
                             dtype=0 if dtype == "f32" else 1) for pad, shift in placements(form)])
        for g in got:
            assert g["rc"] == 0
            kernels = [n for n in g["names"] if not n.startswith("reduce")]
            assert kernels == (["dw_mfma<%d>" % br] if cases is TILES else ["reblock", "dw_mfma<32>"]), (dtype, br, bc, M, K, N)
            assert any(n.startswith("reduce") for n in g["names"]) == splits
            forms = [re.search(r"FormE(\d)", n)[1] for n in g["mangled"] if "dw_mfma_kernel" in n]
            assert forms == [str(("plain", "odd", "packed").index(form))], (dtype, br, bc, M, K, N)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,br,bc,form,splits,M,K,N", TILES + RETILED)
def test_dw_of_single_products_in_tiles(dtype, br, bc, form, splits, M, K, N):
    """Against the oracle, as the other parity tests do: NaN around the rows of dY and behind the values, entries of a block-row in
    order and shuffled, written to and added to a dW with a pitch of its own."""
    rng = np.random.default_rng(M + bc)
    X, dY = rand_pair(M, K, N, dtype, seed=M + K)
    _, o_mask, o_rp, o_ci, o_val = oracle.prune(X, br, bc, 0.6)
    ref = oracle.dw(oracle.mask_dense(X, br, bc, o_mask), dY)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    tol = DW_TOL_DERIVED if dtype == "bf16" else DW_TOL["f32"]
    vals = torch.full((o_val.size + 64,), float("nan"), device="cuda", dtype=dt)
    rp = torch.from_numpy(o_rp).cuda()
    order = np.concatenate([lo + rng.permutation(hi - lo) for lo, hi in zip(o_rp[:-1], o_rp[1:])]).astype(np.int64)
    for pad, shift in placements(form):
        flat = torch.full((shift + M * (N + pad) + 64,), float("nan"), device="cuda", dtype=dt)
        dYd = flat[shift:].as_strided((M, N), (N + pad, 1))
        dYd.copy_(to_dev(dY))
        for pick in (np.arange(len(o_ci)), order):
            val = vals[:o_val.size].view(o_val.shape)
            val.copy_(to_dev(np.ascontiguousarray(o_val[pick]).reshape(-1, bc)).reshape(o_val.shape))
            ci = torch.from_numpy(np.ascontiguousarray(o_ci[pick])).cuda()
            out = torch.full((K, N + 5), 0.25, device="cuda")
            B.bsr_t_dense_matmul(rp, ci, val, M, K, br, bc, dYd, dW=out[:, :N])
            got = out.cpu().numpy()
            assert dw_error(got[:, :N], ref) <= tol and (got[:, N:] == 0.25).all()
            B.bsr_t_dense_matmul(rp, ci, val, M, K, br, bc, dYd, dW=out[:, :N], accumulate=True)
            again = out.cpu().numpy()
            # (at most 64 splits are added one by one, each sum rounded to 2^-24 of no more than the largest result)
            assert dw_error(again[:, :N], 2.0 * got[:, :N].astype(np.float64)) <= 64 * 2.0 ** -24 and (again[:, N:] == 0.25).all()
