"""Scores of large matrices whose rows or block widths are no whole 16-byte vectors."""
import numpy as np
import pytest
import torch

import oracle
from paper_2311_16883_amd import binding as B
from test_gpu_parity import rand_pair, to_dev


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("M,K,br,bc,pad", [
    (1400, 1301, 14, 14, 0),      # rows on odd elements, blocks of a vector and three quarters
    (1393, 1302, 14, 14, 5),      # a last block-row of seven rows, far rows
    (2050, 2001, 32, 32, 0),      # whole vectors in a block, one column in the last block-column
    (3001, 1003, 64, 64, 3),
    (900, 3007, 1, 100, 0),       # 13 vectors on 16 lanes
    (40000, 3, 2, 2, 0),          # a vector reaches over several rows and, for the last ones, beyond the matrix
    (5000, 21, 7, 5, 0),
])
def test_scores_of_rows_at_any_alignment(M, K, br, bc, pad, dtype):
    """Against the oracle, to the rounding of sums of br * bc terms in binary64; alone and in a batch, from the first element of
    a buffer, and from one in the middle of NaN (between the rows, too)."""
    X, _ = rand_pair(M, K, 8, dtype, seed=M + K)
    ref = oracle.prune(X, br, bc, 0.5)[0].reshape(-1)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    flat = torch.full((M * (K + pad) + 64,), float("nan"), device="cuda", dtype=dt)
    Xd = flat[33:].as_strided((M, K), (K + pad, 1))
    Xd.copy_(to_dev(X))
    last = flat[:(M - 1) * (K + pad) + K].clone().as_strided((M, K), (K + pad, 1))    # nothing behind the last element
    last.copy_(Xd)
    got = [B.bsr_score_select(x, br, bc, 0.5, want_scores=True)[1] for x in (Xd, last)]
    nb = -(-M // br) * -(-K // bc)
    scores = [torch.empty(nb, dtype=torch.float64, device="cuda") for _ in range(2)]
    B.bsr_score_select_batched(B.SelectBatch([Xd, last], [(br, bc)] * 2, [0.5] * 2, scores=scores))
    torch.cuda.synchronize()
    for s in got + scores:
        assert np.all(np.abs(s.cpu().numpy().reshape(-1) - ref) <= 2.0 ** -52 * br * bc * ref)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("M,K,br,bc,pad", [
    (5, 3, 2, 2, 0),              # hardly more than a vector in all
    (256, 128, 16, 16, 0),        # whole vectors; the largest that one workgroup takes in binary32
    (100, 321, 14, 14, 0),        # odd rows, vectors beyond blocks and matrix
    (37, 500, 1, 64, 3),
    (127, 130, 64, 64, 1),        # few blocks: 64 lanes for each
    (1000, 31, 7, 5, 0),          # 1001 blocks
    (64, 512, 100, 256, 0),       # one block-row, less than a block high
])
def test_small_matrices_scored_and_selected_by_one_workgroup(M, K, br, bc, pad, dtype):
    """Scores to the rounding of their sums, masks as the oracle's at keeps from none to all, with and without scores asked for."""
    X, _ = rand_pair(M, K, 8, dtype, seed=M + K)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    flat = torch.full((M * (K + pad) + 64,), float("nan"), device="cuda", dtype=dt)
    Xd = flat[33:].as_strided((M, K), (K + pad, 1))
    Xd.copy_(to_dev(X))
    last = flat[:(M - 1) * (K + pad) + K].clone().as_strided((M, K), (K + pad, 1))    # nothing behind the last element
    last.copy_(Xd)
    for keep in (0.0, 0.03, 0.5, 1.0):
        ref, o_mask = oracle.prune(X, br, bc, keep)[:2]
        for x in (Xd, last):
            mask, scores = B.bsr_score_select(x, br, bc, keep, want_scores=True)
            alone = B.bsr_score_select(x, br, bc, keep)
            torch.cuda.synchronize()
            assert np.all(np.abs(scores.cpu().numpy().reshape(-1) - ref.reshape(-1)) <= 2.0 ** -52 * br * bc * ref.reshape(-1))
            assert np.array_equal(mask.cpu().numpy().reshape(-1), o_mask.reshape(-1))
            assert torch.equal(mask, alone)
