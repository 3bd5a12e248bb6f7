"""Scores of large matrices whose rows or block widths are no whole 16-byte vectors."""
import re

import numpy as np
import pytest
import torch

import oracle
from paper_2311_16883_amd import binding as B
from test_dw_dispatch import recorder  # noqa: F401
from test_gpu_parity import rand_pair, to_dev


ANY_ALIGNMENT = [
    (1400, 1301, 14, 14, 0),      # rows on odd elements, blocks of a vector and three quarters
    (1393, 1302, 14, 14, 5),      # a last block-row of seven rows, far rows
    (2050, 2001, 32, 32, 0),      # whole vectors in a block, one column in the last block-column
    (3001, 1003, 64, 64, 3),
    (900, 3007, 1, 100, 0),       # 13 vectors on 16 lanes
    (40000, 3, 2, 2, 0),          # a vector reaches over several rows and, for the last ones, beyond the matrix
    (5000, 21, 7, 5, 0),          # too few blocks for these: plain loads
]


def score_form(got):
    """(elements of a vector, whether at any alignment) of the direct and the LDS body, None for other kernels."""
    m = re.search(r"12score_kernelI[ft]Li(\d)ELb(\d)", got["names"][0])
    return m and (int(m[1]), m[2] == "1")


def test_scores_by_form(recorder):  # noqa: F811
    """Blocks whose rows are one aligned load each, and tall narrow ones, are scored by plain loads; what the tests below give for
    loads at any alignment takes these."""
    def forms(dtype, shapes):
        got = recorder([dict(select=dict(M=M, K=K, br=br, bc=bc, ldx=K + pad, X=(1 << 20) + 33 * (2 if dtype else 4)), dtype=dtype) if shift else
                        dict(select=dict(M=M, K=K, br=br, bc=bc, ldx=K + pad), dtype=dtype) for M, K, br, bc, pad, shift in shapes])
        assert [g["rc"] for g in got] == [0] * len(got)
        return [score_form(g) for g in got]

    narrow = [(25088, 1536, br, bc, pad, False) for br, bc in ((16, 4), (128, 4), (16, 2), (64, 1), (1, 1), (4, 1)) for pad in (0, 8)]
    assert forms(1, narrow) == [(s[3], False) for s in narrow]
    tall = [(25088, 1536, 64, 8, 1, False), (25088, 1536, 128, 4, 1, False), (25088, 1536, 64, 18, 0, False), (25088, 1536, 32, 3, 0, False)]
    assert forms(1, tall) == [(1, False), (1, False), (2, False), (1, False)]
    assert forms(0, [(25088, 768, 64, 1, 0, False), (25088, 768, 128, 2, 4, False), (25088, 768, 64, 30, 0, False)]) == \
        [(1, False), (2, False), (2, False)]
    assert forms(1, [(25088, 1533, *s, 0, False) for s in ((14, 14), (16, 6), (32, 32), (1, 32), (2, 4))]) == [(8, True)] * 5
    below = [(*s, True) for s in ANY_ALIGNMENT]
    assert forms(1, below) == [(8, True)] * 6 + [(1, False)]
    assert forms(0, below) == [(4, True), (4, True), (1, False), (4, True), (4, True), (1, False), (1, False)]


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("M,K,br,bc,pad", ANY_ALIGNMENT)
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
    (256, 128, 16, 16, 0),        # whole vectors; as much as one workgroup takes in binary32
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


ALIKE = [
    (5, 3, 2, 2),
    (256, 128, 16, 16),           # row groups of a vector column; 128 KB in binary32
    (100, 321, 14, 14),           # rows on odd elements
    (100, 322, 14, 14),           # pairs in bfloat16 and binary32
    (300, 84, 14, 14),            # contiguous rows: pieces of a span
    (37, 500, 1, 64),             # row segments: two pieces, or whole vectors
    (250, 128, 1, 32),
    (40, 160, 4, 16),             # few-row blocks of whole vectors
    (127, 130, 64, 64),           # few blocks, the last of two columns
    (1000, 31, 7, 5),             # 1001 blocks
    (64, 512, 100, 256),          # one block-row, less than a block high
    (600, 100, 16, 16),
    (130, 40, 128, 8),            # tall blocks
    (100, 72, 32, 36),            # slices of four elements in bfloat16
    (48, 66, 16, 22),             # ... of two
    (30, 28, 14, 14),             # a span of few blocks
]
ALIKE_PITCHES = [(0, 0), (0, 1), (3, 0), (8, 0)]   # beyond K, and elements in front


@pytest.mark.parametrize("dtype", [0, 1])
def test_small_matrices_reach_every_form_of_one_workgroup(recorder, dtype):  # noqa: F811
    """The matrices of the test below take the one-launch kernel in all its forms, and two launches."""
    calls = [dict(select=dict(M=M, K=K, br=br, bc=bc, ldx=K + pad, X=(1 << 20) + shift * (2 if dtype else 4)), dtype=dtype)
             for M, K, br, bc in ALIKE for pad, shift in ALIKE_PITCHES]
    got = recorder(calls)
    assert [g["rc"] for g in got] == [0] * len(got)
    forms = {re.search(r"kernelI[ft]Li(\d)ELb(\d)", g["names"][0]).groups() for g in got if "score_select_small" in g["names"][0]}
    assert forms == {("1", "0"), ("2", "0"), ("4", "0"), ("4", "1")} if dtype == 0 else \
        {("1", "0"), ("2", "0"), ("4", "0"), ("8", "0"), ("8", "1")}
    assert {len(g["names"]) for g in got} == {1, 2}


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("M,K,br,bc", ALIKE)
def test_small_matrices_rank_alike_in_every_call(M, K, br, bc, dtype):
    """Scores and masks of a matrix, byte for byte: from the single call, among others in a batch, without a workspace, and in
    groups of all block-rows.  Blocks that hold the same values in another order make the mask a matter of the last bit."""
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    rng = np.random.default_rng(M + K)
    nbr, nbc = -(-M // br), -(-K // bc)
    one = rng.standard_normal(br * bc)
    alike = np.stack([rng.permutation(one) for _ in range(nbr * nbc)]).reshape(nbr, nbc, br, bc)
    alike = alike.transpose(0, 2, 1, 3).reshape(nbr * br, nbc * bc)[:M, :K]
    large = torch.randn(3000, 96, device="cuda").to(dt)
    for data in (rng.standard_normal((M, K)), alike):
        for pad, shift in ALIKE_PITCHES:
            flat = torch.zeros(M * (K + pad) + 64, device="cuda", dtype=dt)
            X = flat[shift:].as_strided((M, K), (K + pad, 1))
            X.copy_(torch.from_numpy(data).cuda())
            for keep in (0.3, 0.5):
                mask, scores = B.bsr_score_select(X, br, bc, keep, want_scores=True)
                got = [(B.bsr_score_select(X, br, bc, keep), scores),
                       B.bsr_score_select_grouped(X, br, bc, nbr, keep, want_scores=True),
                       B.bsr_score_select_static(X, br, bc, keep, torch.empty_like(mask), scores=torch.empty_like(scores))]
                for others in (0, 1, 5):
                    out = torch.empty_like(scores)
                    masks = B.bsr_score_select_batched(B.SelectBatch([X] + [large] * others, [(br, bc)] + [(32, 32)] * others,
                                                                     [keep] * (1 + others), scores=[out] + [None] * others))
                    got.append((masks[0], out))
                torch.cuda.synchronize()
                for m, s in got:
                    assert torch.equal(s.view(torch.int64).reshape(-1), scores.view(torch.int64).reshape(-1))
                    assert torch.equal(m.reshape(-1), mask.reshape(-1))
