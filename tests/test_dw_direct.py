"""dW of products on their own whose waves gather the kept blocks: which calls take that kernel (CPU), and its results at the
edges of its tiles, units, splits and lists."""
import numpy as np
import pytest
import torch

import oracle
from paper_2311_16883_amd import binding as B
from test_dw_dispatch import one, recorder  # noqa: F401
from test_gpu_parity import DW_TOL, DW_TOL_DERIVED, dw_error, rand_pair, to_dev


def test_single_products_by_kernel(recorder):  # noqa: F811
    """Alone (single call or a batch of one): products that gain whatever is kept, small ones and such as the 128x128 tiles fill
    badly; not those that would take longer with most blocks kept, wide activations and much to multiply.  Several go as before.
    The queried workspace is enough on both sides of the line."""
    f32, bf16 = 0, 1
    direct = [(f32, 256, 128, 64, 16), (f32, 27601, 228, 192, 14), (f32, 1294, 1344, 1440, 32), (f32, 342, 108, 86, 64),
              (bf16, 256, 128, 64, 16), (bf16, 1202, 152, 446, 32), (bf16, 705, 416, 128, 14), (f32, 25088, 196, 196, 14), (f32, 50176, 196, 196, 14),
              (bf16, 10000, 196, 196, 14), (bf16, 2000, 1000, 190, 16)]
    tiles = [(f32, 12544, 384, 1536, 32), (f32, 6272, 384, 1536, 64), (f32, 13986, 1877, 39, 14), (f32, 12544, 768, 768, 16),
             (f32, 12544, 384, 384, 14), (f32, 50176, 3072, 768, 16), (f32, 1000, 24000, 300, 14), (f32, 4096, 20000, 8, 16),
             (f32, 25842, 42, 464, 32), (f32, 20734, 2592, 64, 64), (bf16, 9947, 411, 1001, 32), (bf16, 7001, 901, 501, 32),
             (bf16, 5615, 96, 2160, 64),
             (bf16, 6272, 384, 1536, 32), (bf16, 4415, 456, 220, 14), (bf16, 8117, 337, 585, 64), (bf16, 49152, 196, 196, 14)]
    for shapes, key in ((direct, "dw_direct"), (tiles, "dw_mfma")):
        alone = [dict(one(*s), dtype=dtype) for dtype, *s in shapes]
        got = recorder(alone + [dict(a, batched=True) for a in alone])
        assert [g["rc"] for g in got] == [0] * len(got)
        assert all(key in g["names"][0] for g in got), got
    segments = [dict(items=[dict(M=M, K=K, N=N, br=1, bc=bc)], dtype=dtype) for dtype in (f32, bf16)
                for M, K, N, bc in ((742, 96, 2848, 64), (13177, 448, 32, 32), (39, 480, 214, 64), (25088, 384, 1536, 32),
                                    (742, 96, 2848, 48), (4096, 10000, 8, 32), (500, 20000, 40, 32), (24, 59, 10, 32))]
    got = recorder(segments + [dict(c, batched=True) for c in segments])
    assert [g["rc"] for g in got] == [0] * 32
    assert ["dw_direct" in g["names"][0] for g in got] == ([True] * 3 + [False] * 5) * 4
    pair = dict(items=one(256, 128, 64, 16)["items"] * 2, batched=True, dtype=f32)
    got = recorder([pair, dict(one(256, 128, 64, 16, values=(1 << 20) + 4), dtype=f32), one(256, 128, 64, 16, values=(1 << 20) + 2)])
    assert ["dw_direct" in g["names"][0] for g in got] == [False, True, False]


def test_products_gathered_by_the_waves_need_no_workspace_of_their_own(recorder):  # noqa: F811
    """The query names what the other kernels need (re-tiled row segments: the copy and its partial sums), whichever takes the
    product; it is enough on either side of the line."""
    segments = [((5232, 4516, 6468, 32), 47 << 20), ((5545, 573, 7444, 96), 7 << 20), ((4534, 3042, 3895, 64), 28 << 20)]
    got = recorder([dict(items=[dict(M=M, K=K, N=N, br=1, bc=bc)]) for (M, K, N, bc), _ in segments])
    assert [g["rc"] for g in got] == [0] * 3 and all("reblock" in g["names"][0] for g in got)
    assert all(g["ws"] <= most for g, (_, most) in zip(got, segments)), [g["ws"] for g in got]
    for dtype in (0, 1):
        for br, bc in ((14, 14), (16, 16), (32, 32), (1, 32), (1, 96)):
            for K, N in ((64, 64), (196, 196), (411, 1001), (1500, 24)):
                got = recorder([dict(items=[dict(M=M, K=K, N=N, br=br, bc=bc)], dtype=dtype) for M in range(100, 30000, 700)])
                assert [g["rc"] for g in got] == [0] * len(got)


@pytest.mark.gpu
@pytest.mark.parametrize("b", [14, 16, 32, 64])
@pytest.mark.parametrize("M,K,N,keep,dtype", [
    (1, 1, 1, 1.0, "f32"),
    (65, 67, 33, 0.5, "f32"),            # ragged rows, a strip and a tile of dY in part
    (500, 130, 257, 0.3, "f32"),         # beyond two tiles of 128 columns by one
    (2500, 40, 66, 0.9, "f32"),          # many units for each of 16 waves
    (14400, 33, 5, 0.2, "f32"),          # 14x14: more block-rows than the list of one split holds
    (6000, 96, 200, 0.7, "f32"),         # several splits
    (1, 1, 8, 1.0, "bf16"),
    (65, 67, 34, 0.5, "bf16"),
    (65, 67, 33, 0.5, "bf16"),           # rows on odd elements
    (500, 130, 257, 0.3, "bf16"),
    (2500, 40, 66, 0.9, "bf16"),
    (700, 500, 131, 0.6, "bf16"),
    (500, 40, 2001, 0.4, "bf16"),        # tiles of 128 columns
    (16000, 200, 45, 0.75, "bf16"),      # several splits, and more block-rows than the list of one holds
])
def test_dw_of_blocks_gathered_by_the_waves(M, K, N, keep, dtype, b):
    """Against the oracle: NaN around the rows of dY, pitches of 0 and 1 beyond N, NaN behind the stored blocks, entries of a
    block-row in order and shuffled, written to and added to a dW with a pitch of its own whose padding stays as it is."""
    rng = np.random.default_rng(M + b)
    X, dY = rand_pair(M, K, N, dtype, seed=M + K)
    _, o_mask, o_rp, o_ci, o_val = oracle.prune(X, b, b, keep)
    ref = oracle.dw(oracle.mask_dense(X, b, b, o_mask), dY)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    flat = torch.full((M * (N + 3) + 128,), float("nan"), device="cuda", dtype=dt)
    vals = torch.full((o_val.size + 64,), float("nan"), device="cuda", dtype=dt)
    rp = torch.from_numpy(o_rp).cuda()
    order = np.concatenate([lo + rng.permutation(hi - lo) for lo, hi in zip(o_rp[:-1], o_rp[1:])]).astype(np.int64)
    for pick, shift, pad in ((np.arange(len(o_ci)), 64, 0), (order, 65, 1), (order, 64, 2)):
        flat.fill_(float("nan"))
        dYd = flat[shift:].as_strided((M, N), (N + pad, 1))
        dYd.copy_(to_dev(dY))
        val = vals[:o_val.size].view(o_val.shape)
        val.copy_(to_dev(np.ascontiguousarray(o_val[pick]).reshape(-1, b)).reshape(o_val.shape))
        ci = torch.from_numpy(np.ascontiguousarray(o_ci[pick])).cuda()
        out = torch.full((K, N + 5), 0.25, device="cuda")
        B.bsr_t_dense_matmul(rp, ci, val, M, K, b, b, dYd, dW=out[:, :N])
        got = out.cpu().numpy()
        assert dw_error(got[:, :N], ref) <= (DW_TOL_DERIVED if dtype == "bf16" else DW_TOL["f32"])
        assert (got[:, N:] == 0.25).all()
        B.bsr_t_dense_matmul(rp, ci, val, M, K, b, b, dYd, dW=out[:, :N], accumulate=True)
        again = out.cpu().numpy()
        # (at most 64 splits are added one by one, each sum rounded to 2^-24 of no more than the largest result)
        assert dw_error(again[:, :N], 2.0 * got[:, :N].astype(np.float64)) <= 64 * 2.0 ** -24 and (again[:, N:] == 0.25).all()


@pytest.mark.gpu
@pytest.mark.parametrize("bc", [32, 96])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("M,K,N,keep", [
    (1, 1, 8, 1.0),
    (37, 130, 33, 0.5),           # rows on odd elements, a segment in part, units in part
    (4097, 40, 34, 0.7),          # one row more than the list of a split holds
    (900, 1000, 140, 0.02),       # strips that keep nothing
    (1200, 700, 257, 1.0),        # every row
])
def test_dw_of_row_segments_gathered_by_the_waves(M, K, N, keep, dtype, bc):
    """As above, in 1 x bc blocks."""
    rng = np.random.default_rng(M + bc)
    X, dY = rand_pair(M, K, N, dtype, seed=M + K)
    _, o_mask, o_rp, o_ci, o_val = oracle.prune(X, 1, bc, keep)
    ref = oracle.dw(oracle.mask_dense(X, 1, bc, o_mask), dY)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    flat = torch.full((M * (N + 3) + 128,), float("nan"), device="cuda", dtype=dt)
    vals = torch.full((o_val.size + 64,), float("nan"), device="cuda", dtype=dt)
    rp = torch.from_numpy(o_rp).cuda()
    order = np.concatenate([lo + rng.permutation(hi - lo) for lo, hi in zip(o_rp[:-1], o_rp[1:])]).astype(np.int64)
    for pick, shift, pad in ((np.arange(len(o_ci)), 64, 0), (order, 65, 1)):
        flat.fill_(float("nan"))
        dYd = flat[shift:].as_strided((M, N), (N + pad, 1))
        dYd.copy_(to_dev(dY))
        val = vals[:o_val.size].view(o_val.shape)
        val.copy_(to_dev(np.ascontiguousarray(o_val[pick]).reshape(-1, bc)).reshape(o_val.shape))
        ci = torch.from_numpy(np.ascontiguousarray(o_ci[pick])).cuda()
        got = B.bsr_t_dense_matmul(rp, ci, val, M, K, 1, bc, dYd).cpu().numpy()
        assert dw_error(got, ref) <= (DW_TOL_DERIVED if dtype == "bf16" else DW_TOL["f32"])
        dead = np.ones(K, bool)
        for j in np.unique(o_ci):
            dead[j * bc:(j + 1) * bc] = False
        assert not got[dead].any()
