"""Which kernels a dW call would launch, and with what workspace: the host code runs against a recorder of launches
(tests/launch_recorder.c), at sizes that need no memory here.  CPU only."""
import json
import random
import re
import subprocess
import sys
from pathlib import Path

import pytest

import test_gpu_parity as parity
from paper_2311_16883_amd import binding as B

HERE = Path(__file__).resolve().parent
LIB = HERE.parent / "paper_2311_16883_amd" / "libbsr_actprune.so"


@pytest.fixture(scope="module")
def recorder(tmp_path_factory):
    so = tmp_path_factory.mktemp("recorder") / "liblaunch_recorder.so"
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-o", str(so), str(HERE / "launch_recorder.c")], check=True)
    B.lib()                                  # built if it is not there yet

    def record(calls, lib=LIB):
        """Per call: return code, queried workspace, launched kernels as "name<leading template arguments>"."""
        r = subprocess.run([sys.executable, str(HERE / "recorded_calls.py"), str(so), str(lib)], input=json.dumps(calls),
                           capture_output=True, text=True, timeout=300)
        assert r.returncode == 0, r.stderr
        got = json.loads(r.stdout)
        for g in got:
            g["mangled"] = [n for n, _ in g["kernels"]]
            g["kernels"] = [(kernel_name(n), w) for n, w in g["kernels"]]
            g["names"] = [n for n, _ in g["kernels"]]
        return got

    return record


def kernel_name(mangled):
    """dw_wide<16>, dw_mfma<16>, dw_narrow<7>, dw_generic, reblock, reduce, reduce_shared, from the mangled names."""
    for key, name in (("dw_wide_batched_kernel", "dw_wide"), ("dw_mfma_batched_kernel", "dw_mfma"), ("dw_mfma_kernel", "dw_mfma"),
                      ("dw_narrow_batched_kernel", "dw_narrow")):
        if key in mangled:
            return "%s<%s>" % (name, re.search(r"Li(\d+)E", mangled).group(1))
    for key, name in (("dw_generic_kernel", "dw_generic"), ("reblock_kernel", "reblock"),
                      ("splitk_reduce_shared", "reduce_shared"), ("splitk_reduce", "reduce")):
        if key in mangled:
            return name
    return mangled


def one(M, K, N, b, **more):
    return {"items": [dict(M=M, K=K, N=N, b=b, **more)]}


def batch(*items):
    return {"items": [dict(zip("MKNb", it)) if isinstance(it, tuple) else it for it in items], "batched": True}


def products(got):
    return [n for n in got["names"] if not n.startswith("reduce")]


def reductions(got):
    return [n for n in got["names"] if n.startswith("reduce")]


@pytest.mark.parametrize("M,K,N,other", [(4000, 300000, 8, "dw_wide<16>"), (4096, 270000, 8, "dw_wide<16>"),
                                         (2900000, 384, 384, "dw_generic"), (1 << 20, 1024, 8, "dw_generic")])
@pytest.mark.parametrize("copies", [1, 2])
def test_batched_dw_beyond_2_gib_is_not_given_to_the_kernel_that_cannot_address_it(recorder, M, K, N, other, copies):
    """16x16 blocks of 2 GiB and more, too little to multiply (or too few tiles) for the wide tiles: the 128x128 kernel takes
    offsets from 2 GiB on for "pruned".  The wide tiles multiply them all the same if they are enough to fill the GPU, else
    the general kernel."""
    got, = recorder([batch(*[(M, K, N, 16)] * copies)])
    assert got["rc"] == 0
    assert products(got) == ([other] if other == "dw_wide<16>" else [other] * copies)


def operands_below(M, K, b, gib):
    """Stored blocks, all kept, in bytes: below gib GiB?"""
    return -(-M // b) * -(-K // b) * b * b * 2 < gib << 30


@pytest.mark.parametrize("b", [16, 32, 64])
def test_dw_calls_with_the_queried_workspace_are_taken(recorder, b):
    """Activations around 2 GiB, where the 128x128 tiles end, and 4 GiB, where the wide tiles end, alone and in batches of two:
    exactly the workspace that the query names is enough, whatever kernel the call takes."""
    shapes = [(700000, 1536, 1536), (1500000, 768, 768), (1000000, 1536, 512), (400000, 3072, 768), (350000, 3072, 768),
              (349000, 3072, 768), (699000, 1536, 1536), (698000, 3072, 768), (700000, 3072, 768), (2900000, 384, 384),
              (4000, 300000, 8), (4000, 300000, 1024), (1 << 20, 1024, 8), (1 << 20, 1024, 136), (5000000, 400, 136)]
    single = recorder([one(M, K, N, b) for M, K, N in shapes])
    pairs = recorder([batch((M, K, N, b), (M, K, N, b)) for M, K, N in shapes])
    mixed = recorder([batch((M, K, N, b), (6272, 384, 1536, b)) for M, K, N in shapes])
    assert [g["rc"] for g in single + pairs + mixed] == [0] * 3 * len(shapes)
    kernels = {n for g in single for n in g["names"]}
    assert {f"dw_wide<{b}>", "dw_generic"} <= kernels
    for (M, K, N), g in zip(shapes, single):
        if not operands_below(M, K, b, 2):
            assert "dw_mfma<%d>" % b not in g["names"]
        if not operands_below(M, K, b, 4):
            assert products(g) == ["dw_generic"]


@pytest.mark.parametrize("b", [32, 64])
def test_dw_with_a_pitch_of_dy_that_only_the_wide_tiles_can_address(recorder, b):
    """Too little to multiply for the wide tiles, but rows of dY so far apart that the 128x128 tiles cannot take them: the
    matrix cores all the same, alone and in batches."""
    far = dict(M=1000, K=1000, N=4000, b=b, lddy=1600000)
    near = dict(far, M=200, lddy=4000)
    single, pair, both, plain = recorder([{"items": [far]}, batch(far, far), batch(far, near), {"items": [near]}])
    assert [g["rc"] for g in (single, pair, both, plain)] == [0] * 4
    assert products(single) == products(pair) == [f"dw_wide<{b}>"]
    assert sorted(products(both)) == [f"dw_mfma<{b}>", f"dw_wide<{b}>"]
    assert products(plain) == [f"dw_mfma<{b}>"]


def test_batched_dw_lines_of_the_wide_tiles_go_by_block_size(recorder):
    """Products of different block sizes don't share a launch, so they don't lend each other work: each size goes where it
    would go by itself.  32x32 and 64x64 blocks lend each other tiles."""
    large, little, small = (25088, 384, 1536, 32), (3136, 384, 1536, 16), (6272, 384, 1536, 64)
    alone = [products(g) for g in recorder([batch(large), batch(little), batch(small)])]
    assert alone == [["dw_wide<32>"], ["dw_mfma<16>"], ["dw_mfma<64>"]]
    got, = recorder([batch(large, little, small)])
    assert got["rc"] == 0 and sorted(products(got)) == sorted(sum(alone, []))
    half = [(14600, 384, 896, b) for b in (16, 32, 64)]
    assert [products(g) for g in recorder([batch(h) for h in half])] == [["dw_mfma<16>"], ["dw_mfma<32>"], ["dw_mfma<64>"]]
    assert sorted(products(recorder([batch(*half)])[0])) == ["dw_mfma<16>", "dw_wide<32>", "dw_wide<64>"]


@pytest.mark.parametrize("b", [32, 64])
def test_dw_line_of_the_wide_tiles_counts_whole_tiles_of_the_other_kernel(recorder, b):
    """A product on its own goes to the wide tiles by what the 128x128 tiles would multiply, whatever part of a tile dW fills;
    several by what there is to multiply."""
    wide = [(8147, 152, 1968), (4062, 416, 2128), (12544, 1536, 256), (9877, 128, 3816), (25088, 384, 1536)]
    narrow = [(6272, 384, 1536), (800, 2048, 2048), (3677, 760, 1208), (3591, 1952, 224), (1095, 1240, 2832), (10098, 3616, 32)]
    assert [products(g) for g in recorder([one(*s, b) for s in wide])] == [[f"dw_wide<{b}>"]] * len(wide)
    assert [products(g) for g in recorder([batch((*s, b)) for s in wide])] == [[f"dw_wide<{b}>"]] * len(wide)
    assert [products(g) for g in recorder([one(*s, b) for s in narrow])] == [[f"dw_mfma<{b}>"]] * len(narrow)
    got = recorder([batch((8147, 152, 1968, b), (8147, 152, 1968, b)), batch((3591, 1952, 224, b), (8147, 152, 2500, b))])
    assert [products(g) for g in got] == [[f"dw_mfma<{b}>"], [f"dw_mfma<{b}>"]]
    assert products(recorder([batch((8147, 152, 1968, b), (8147, 152, 2200, b))])[0]) == [f"dw_wide<{b}>"]


def test_dw_of_16x16_blocks_takes_wide_tiles_where_they_are_filled(recorder):
    """Alone and in batches: work enough, and tiles that fit dW and keep the compute units busy not much worse than 128x128 tiles."""
    wide = [(50176, 1536, 384), (12348, 768, 3072), (40000, 1500, 1000), (49224, 3160, 264)]
    narrow = [(27817, 408, 3440), (11825, 1576, 1664), (30734, 464, 1816), (6867, 2944, 2528), (25088, 1536, 384)]
    assert [products(g) for g in recorder([one(*s, 16) for s in wide])] == [["dw_wide<16>"]] * len(wide)
    assert [products(g) for g in recorder([one(*s, 16) for s in narrow])] == [["dw_mfma<16>"]] * len(narrow)
    even = batch(*[(4116, 768, 3072, 16)] * 18)
    uneven = batch((33324, 352, 200, 16), (14904, 2880, 112, 16), (17969, 688, 128, 16), (22727, 1344, 72, 16), (13016, 1824, 2232, 16))
    many = batch(*[(6272, 384, 1536, 16)] * 30)        # more than one launch holds
    assert [products(g)[:1] for g in recorder([even, uneven, many])] == [["dw_wide<16>"], ["dw_mfma<16>"], ["dw_wide<16>"]]


def test_dw_reductions_are_shared_for_small_matrices_only_and_in_one_launch(recorder):
    """Threads share an output of many splits while there are few outputs; the products of a launch are added up together."""
    calls = [one(50176, 196, 196, 14), one(50176, 300, 301, 16), one(50176, 512, 512, 14), one(25088, 384, 768, 32),
             batch((6272, 384, 384, 14), (25088, 384, 384, 14)), batch((700, 140, 332, 32), (25088, 100, 36, 32)),
             batch((25088, 384, 1536, 32), (25088, 196, 196, 14), (25088, 196, 196, 14))]
    assert [reductions(g) for g in recorder(calls)] == [["reduce_shared"], ["reduce_shared"], ["reduce"], ["reduce"], ["reduce"],
                                                        ["reduce_shared"], ["reduce"]]


def partials(M, K, N, splits):
    return splits * K * N * 4


def test_dw_workspace_of_the_wide_tiles(recorder):
    """Sixteen splits, more only where the contraction is long enough to be split further: 1.09 GB for the 36 products of
    ResMLP-S12 at batch 128.  What is enough for a batch is enough for a shorter one and for a part of it."""
    fc1, fc2, patches = (25088, 384, 1536), (50176, 1536, 384), (49152, 196, 196)
    for b in (32, 64):
        got = recorder([one(*fc1, b), one(*fc2, b)])
        assert [g["ws"] for g in got] == [partials(*fc1, 16), partials(*fc2, 21)]
        assert [g["kernels"][0] for g in got] == [(f"dw_wide<{b}>", 16 * 12), (f"dw_wide<{b}>", 256)]
    for b in (16, 32, 64):
        layers = [x for _ in range(12) for x in ((*patches, 14), (*fc1, b), (25088, 1536, 384, b))]
        network, part, short = recorder([batch(*layers), batch(*layers[:7]), batch(*[(M // 3, K, N, b) for M, K, N, b in layers])])
        assert network["rc"] == 0 and network["kernels"][0] == (f"dw_wide<{b}>", 512)   # 21 tile by tile, three split
        assert network["ws"] == sum(g["ws"] for g in recorder([one(*x) for x in layers])) < 1090 << 20
        assert part["ws"] < network["ws"] and short["ws"] <= network["ws"]
        sizes = [g["ws"] for g in recorder([one(M, *shape, b) for shape in ((384, 1536), (1536, 384), (1536, 256), (200, 2000))
                                            for M in range(196, 196 * 300, 196)])]
        for k in range(0, len(sizes), 299):
            assert sizes[k:k + 299] == sorted(sizes[k:k + 299])


def test_batched_dw_is_taken_whatever_the_operands_allow(recorder):
    """The workspace is sized for aligned operands and contiguous rows; products that are neither take other kernels, or split
    less, and their companions too.  None is refused."""
    rng = random.Random(3)
    calls = []
    for _ in range(300):
        items = []
        for _ in range(rng.randint(1, 30 if rng.random() < 0.1 else 5)):
            M, K, N = (int(2 ** rng.uniform(*r)) for r in ((4, 16), (3, 12), (3, 12)))
            b = rng.choice((14, 16, 16, 32, 32, 64, 8))
            unit = rng.choice((1, 8, 8))
            N = max(unit, N // unit * unit)
            items.append(dict(M=M, K=K, N=N, b=b, lddy=rng.choice((N, N, N + 8, N + 3, 200000)), lddw=N + rng.choice((0, 1)),
                              values=(1 << 20) + rng.choice((0, 0, 2)), dY=(1 << 20) + rng.choice((0, 0, 2, 4)),
                              accumulate=rng.choice((0, 1))))
        calls.append({"items": items, "batched": True})
    assert [g["rc"] for g in recorder(calls)] == [0] * len(calls)


def test_the_gpu_tests_of_the_wide_tiles_reach_them(recorder):
    """The sizes that the GPU tests give for the wide tiles, and for both sides of their lines, take the kernels they name."""
    for b in (32, 64):
        for M, K, N in (parity.WIDE_RAGGED, parity.WIDE_NON_FINITE):
            got, = recorder([one(M, K, N, b)])
            assert products(got) == [f"dw_wide<{b}>"]
    shapes = [s[:4] for s in parity.wide_random_shapes()]
    assert [products(g) for g in recorder([one(*s) for s in shapes])] == [[f"dw_wide<{s[3]}>"] for s in shapes]
    assert products(recorder([batch(*shapes)])[0]) == ["dw_wide<32>", "dw_wide<64>"]
    alone = recorder([one(*c[:4]) for c in parity.LARGE_DW])
    pairs = recorder([batch(c[:4], c[:4]) for c in parity.LARGE_DW])
    assert [products(g) for g in alone] == [[f"dw_{c[5]}<{c[3]}>"] for c in parity.LARGE_DW]
    assert [products(g) for g in pairs] == [[f"dw_{c[6]}<{c[3]}>"] for c in parity.LARGE_DW]
    for b in (16, 32, 64):                  # split products and such as one workgroup runs whole
        assert {bool(reductions(g)) for c, g in zip(parity.LARGE_DW, alone) if c[3] == b and c[5] == "wide"} == {False, True}
    for b in (16, 32, 64):
        far, near = dict(M=1000, K=1000, N=400, b=b, lddy=1600000), dict(M=1000, K=1000, N=400, b=b)
        got = recorder([{"items": [far]}, batch(far, near, far)])
        assert [sorted(products(g)) for g in got] == [[f"dw_wide<{b}>"], [f"dw_mfma<{b}>", f"dw_wide<{b}>"]]
    tiles, = recorder([batch(*[(16000, 1536, 512, 32)] * 24)])
    assert tiles["kernels"][0][0] == "dw_wide<32>" and reductions(tiles) == ["reduce"]
