"""dW of products on their own whose waves gather the kept blocks: which calls take that kernel (CPU), and its results at the
edges of its tiles, units, splits and lists."""
import re

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
    (500, 40, 2001, 0.4, "bf16"),        # many tiles of dY, one column in the last
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


# One product for every form of the kernel that a call of its own can take: element, rows of a block, waves of a workgroup (4: tiles
# of 128 columns, 8: 64, 16: 32), rows of dY on odd elements, splits; M, K, N, and the columns of a block.
FORMS = [
    ("f32", 1, 4, False, False, 23, 893, 586, 96), ("f32", 1, 4, False, True, 1855, 1092, 78, 96),
    ("f32", 1, 8, False, False, 66, 9, 4, 32), ("f32", 1, 8, False, True, 1259, 12, 4, 32),
    ("f32", 1, 16, False, False, 267, 33, 4, 32), ("f32", 1, 16, False, True, 17222, 8, 5, 32),
    ("f32", 14, 4, False, False, 24, 1876, 96, 14), ("f32", 14, 4, False, True, 4453, 394, 68, 14),
    ("f32", 14, 8, False, False, 23, 1825, 50, 14), ("f32", 14, 8, False, True, 2426, 40, 746, 14),
    ("f32", 14, 16, False, False, 20, 9, 10, 14), ("f32", 14, 16, False, True, 1422, 11, 6, 14),
    ("f32", 16, 4, False, False, 28, 720, 348, 16), ("f32", 16, 4, False, True, 2122, 575, 232, 16),
    ("f32", 16, 8, False, False, 20, 267, 508, 16), ("f32", 16, 8, False, True, 3211, 566, 38, 16),
    ("f32", 16, 16, False, False, 25, 9, 6, 16), ("f32", 16, 16, False, True, 2448, 8, 6, 16),
    ("f32", 32, 4, False, False, 28, 810, 624, 32), ("f32", 32, 4, False, True, 5907, 389, 230, 32),
    ("f32", 32, 8, False, False, 40, 8, 5, 32), ("f32", 32, 8, False, True, 1111, 25, 4, 32),
    ("f32", 32, 16, False, False, 77, 9, 4, 32), ("f32", 32, 16, False, True, 6520, 11, 4, 32),
    ("f32", 64, 4, False, False, 20, 576, 1068, 64), ("f32", 64, 8, False, False, 49, 12, 4, 64),
    ("f32", 64, 8, False, True, 1196, 10, 8, 64), ("f32", 64, 16, False, False, 75, 11, 4, 64),
    ("f32", 64, 16, False, True, 6216, 16, 4, 64), ("bf16", 1, 4, False, False, 21, 1677, 288, 32),
    ("bf16", 1, 4, False, True, 3676, 730, 94, 32), ("bf16", 1, 4, True, False, 22, 970, 557, 32),
    ("bf16", 1, 8, False, False, 21, 79, 2754, 96), ("bf16", 1, 8, False, True, 11449, 9, 380, 32),
    ("bf16", 1, 8, True, False, 20, 1548, 199, 96), ("bf16", 1, 8, True, True, 3261, 500, 33, 32),
    ("bf16", 1, 16, False, False, 183, 8, 4, 96), ("bf16", 1, 16, False, True, 4541, 47, 4, 32),
    ("bf16", 1, 16, True, False, 216, 11, 5, 96), ("bf16", 1, 16, True, True, 5248, 34, 5, 96),
    ("bf16", 14, 4, False, False, 23, 285, 906, 14), ("bf16", 14, 4, False, True, 7672, 209, 214, 14),
    ("bf16", 14, 4, True, False, 31, 1961, 95, 14), ("bf16", 14, 8, False, False, 20, 279, 408, 14),
    ("bf16", 14, 8, False, True, 9722, 15, 228, 14), ("bf16", 14, 8, True, False, 21, 39, 2955, 14),
    ("bf16", 14, 8, True, True, 12076, 141, 63, 14), ("bf16", 14, 16, False, False, 22, 9, 12, 14),
    ("bf16", 14, 16, False, True, 3777, 9, 6, 14), ("bf16", 14, 16, True, False, 25, 10, 5, 14),
    ("bf16", 14, 16, True, True, 5501, 21, 5, 14), ("bf16", 16, 4, False, False, 26, 1136, 194, 16),
    ("bf16", 16, 4, False, True, 16253, 235, 72, 16), ("bf16", 16, 4, True, False, 21, 124, 2953, 16),
    ("bf16", 16, 8, False, False, 20, 569, 238, 16), ("bf16", 16, 8, False, True, 8166, 18, 362, 16),
    ("bf16", 16, 8, True, False, 25, 543, 307, 16), ("bf16", 16, 8, True, True, 7333, 23, 589, 16),
    ("bf16", 16, 16, False, False, 23, 9, 4, 16), ("bf16", 16, 16, False, True, 5300, 8, 6, 16),
    ("bf16", 16, 16, True, False, 23, 47, 5, 16), ("bf16", 16, 16, True, True, 10286, 8, 9, 16),
    ("bf16", 32, 4, False, False, 22, 377, 1372, 32), ("bf16", 32, 4, True, False, 136, 838, 639, 32),
    ("bf16", 32, 8, False, False, 25, 167, 1546, 32), ("bf16", 32, 8, False, True, 6389, 15, 1172, 32),
    ("bf16", 32, 8, True, False, 21, 467, 553, 32), ("bf16", 32, 16, False, False, 27, 10, 4, 32),
    ("bf16", 32, 16, False, True, 7163, 8, 4, 32), ("bf16", 32, 16, True, False, 30, 12, 5, 32),
    ("bf16", 32, 16, True, True, 13036, 9, 5, 32), ("bf16", 64, 4, False, False, 85, 967, 544, 64),
    ("bf16", 64, 8, False, False, 23, 229, 1122, 64), ("bf16", 64, 8, False, True, 5211, 16, 944, 64),
    ("bf16", 64, 8, True, False, 71, 1464, 207, 64), ("bf16", 64, 16, False, False, 24, 11, 6, 64),
    ("bf16", 64, 16, False, True, 5353, 10, 4, 64), ("bf16", 64, 16, True, False, 23, 13, 7, 64),
    ("bf16", 64, 16, True, True, 8725, 17, 9, 64),
]


def form_reached(got):
    m = re.search(r"dw_direct_kernelI([ft])Li(\d+)ELi\d+ELi\d+ELi(\d+)ELi\d+ELi\d+ELb(\d)", got["mangled"][0])
    return m and ("f32" if m[1] == "f" else "bf16", int(m[2]), int(m[3]), m[4] == "1", len(got["names"]) > 1)


def test_the_sizes_above_reach_every_form(recorder):  # noqa: F811
    got = recorder([dict(items=[dict(M=M, K=K, N=N, br=br, bc=bc)], dtype=0 if dtype == "f32" else 1)
                    for dtype, br, _, _, _, M, K, N, bc in FORMS])
    assert [g["rc"] for g in got] == [0] * len(got)
    assert [form_reached(g) for g in got] == [f[:5] for f in FORMS]
    every = {("f32", br, waves, False) for br in (1, 14, 16, 32, 64) for waves in (4, 8, 16)}
    every |= {("bf16", br, waves, odd) for br in (1, 14, 16, 32, 64) for waves in (4, 8, 16) for odd in (False, True)}
    # (wide tiles of 64x64 blocks beside odd rows: no product was found whose plan has them)
    assert {f[:4] for f in FORMS} == every - {("bf16", 64, 4, True)}


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,br,waves,odd,splits,M,K,N,bc", FORMS)
def test_dw_by_every_form_of_the_gathering_waves(dtype, br, waves, odd, splits, M, K, N, bc):
    if br == 1:
        test_dw_of_row_segments_gathered_by_the_waves(M, K, N, 0.6, dtype, bc)
    else:
        test_dw_of_blocks_gathered_by_the_waves(M, K, N, 0.6, dtype, br)
