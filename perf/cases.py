"""Performance cases: the calls that a program makes which trains with pruned activations.

A training program of this library does, for every linear layer, two things per step:
on the way forward it ranks the blocks of the layer's input, keeps the best and stores
them as BSR (``bsr_score_select``, ``bsr_compress``); on the way back it forms the weight
gradient from that BSR tensor (``bsr_t_dense_matmul``).  It does so layer by layer
(kind "train": one layer through the single calls), or for the layers of a whole network
through the batched calls (kinds "prune_set", "grad_set", and "restore_set" for programs
that need the dense masked activation back).  Kind "sample" is the paper's per-sample
ranking followed by the scale gradient of the affine layer.

Inputs are synthetic activations of the shapes the repository's workloads name:
standard normal (what follows a normalisation), GELU of standard normal (what follows
the first MLP layer), output gradients of standard deviation 1e-3.
"""
import math

import torch

from paper_2311_16883_amd import binding as B

DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16}
PATCHES = 196


def listed():
    return [
        # the smallest call: one small layer (a toy model, a classifier head); launches and host work count
        dict(name="tiny_f32_16x16", kind="train", dtype="f32", M=256, K=128, N=64, br=16, bc=16, keep=0.5, dist="gelu"),
        # cross-patch layer of ResMLP-S12 at batch 128, 14x14 blocks over the patch axis, layer by layer
        dict(name="s12_xpatch_14x14", kind="train", dtype="bf16", M=128 * 384, K=PATCHES, N=PATCHES, br=14, bc=14,
             keep=0.5, dist="normal"),
        # first MLP layer of ResMLP-S12 at batch 128, layer by layer: the ordinary call
        dict(name="s12_fc1_32x32", kind="train", dtype="bf16", M=128 * PATCHES, K=384, N=1536, br=32, bc=32, keep=0.5,
             dist="normal"),
        # the same layer in the paper's own precision, batch 64
        dict(name="s12_fc1_f32_32x32", kind="train", dtype="f32", M=64 * PATCHES, K=384, N=1536, br=32, bc=32, keep=0.5,
             dist="normal"),
        # second MLP layer of ResMLP-S24 at batch 256 with the smallest blocks of its sweep and few of them kept
        dict(name="s24_fc2_16x16", kind="train", dtype="bf16", M=256 * PATCHES, K=1536, N=384, br=16, bc=16, keep=0.25,
             dist="gelu"),
        # second MLP layer of ResMLP-B24 at batch 256, 64x64 blocks, a tenth of the channels five times as large
        dict(name="b24_fc2_64x64", kind="train", dtype="bf16", M=256 * PATCHES, K=3072, N=768, br=64, bc=64, keep=0.5,
             dist="hot"),
        # row segments (the block shape of the paper's index overheads) on the first MLP layer
        dict(name="s12_fc1_rows_1x32", kind="train", dtype="bf16", M=128 * PATCHES, K=384, N=1536, br=1, bc=32, keep=0.5,
             dist="normal"),
        # sizes that fit nothing: a short last batch, widths that are no multiple of a vector
        dict(name="ragged_32x32", kind="train", dtype="bf16", M=9947, K=411, N=1001, br=32, bc=32, keep=0.5, dist="gelu"),
        # per-sample ranking (groups of eight samples = 49 block-rows) and the affine layer's scale gradient
        dict(name="s12_affine_per_sample", kind="sample", dtype="bf16", M=128 * PATCHES, K=384, br=32, bc=32,
             group_rows=49, keep=0.5, dist="normal"),
        # all 36 linear-layer inputs of ResMLP-S12 at batch 128, one batched call per stage: forward side,
        dict(name="s12_set_prune", kind="prune_set", dtype="bf16", layers=12, batch=128, dim=384, b=32, keep=0.5),
        # ... the dense masked activations back,
        dict(name="s12_set_restore", kind="restore_set", dtype="bf16", layers=12, batch=128, dim=384, b=32, keep=0.5),
        # ... and the 36 weight gradients
        dict(name="s12_set_grad", kind="grad_set", dtype="bf16", layers=12, batch=128, dim=384, b=32, keep=0.5),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _width(rng, lo, hi):
    """A matrix width: a third of them whole 32s, a third whole 8s, a third anything."""
    n = _log_int(rng, lo, hi)
    unit = rng.choice((32, 8, 1))
    return max(unit, n // unit * unit)


def draw(rng):
    """One more layer or set of layers.  Bounded by the largest listed cases: 400 MB of operands and 120 GFLOP (20 in
    binary32) per layer, the listed sets for the sets."""
    kind = rng.choice(("train", "train", "train", "train", "sample", "prune_set", "restore_set", "grad_set"))
    keep = rng.choice((0.1, 0.25, 0.5, 0.75, 0.9))
    if kind.endswith("_set"):
        dim = rng.choice((192, 384, 768))
        batch = _log_int(rng, 4, 128 if dim <= 384 else 64)
        layers = rng.randint(2, 12)
        if batch * dim * layers > 128 * 384 * 12:
            layers = max(2, 128 * 384 * 12 // (batch * dim))
        return dict(kind=kind, dtype="bf16", layers=layers, batch=batch, dim=dim, b=rng.choice((16, 32, 64)), keep=keep)
    dtype = rng.choice(("bf16", "bf16", "f32"))
    size = 2 if dtype == "bf16" else 4
    while True:
        M, K = _log_int(rng, 200, 50176), _width(rng, 64, 3072)
        if kind == "sample":
            br = bc = rng.choice((14, 16, 32))
            if M * K * size <= 200e6:
                return dict(kind=kind, dtype=dtype, M=M, K=K, br=br, bc=bc, group_rows=rng.randint(7, 56), keep=keep,
                            dist=rng.choice(("normal", "gelu")))
            continue
        N = _width(rng, 32, 3072)
        br, bc = rng.choice(((14, 14), (16, 16), (32, 32), (32, 32), (64, 64), (64, 64), (1, 32), (1, 64)))
        if M * (K + N) * size <= 400e6 and 2.0 * M * K * N <= (120e9 if dtype == "bf16" else 20e9):
            return dict(kind=kind, dtype=dtype, M=M, K=K, N=N, br=br, bc=bc, keep=keep,
                        dist=rng.choice(("normal", "gelu", "hot")))


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _activation(gen, M, K, dist, dtype):
    x = torch.randn(M, K, generator=gen, device="cuda")
    if dist != "normal":
        x = torch.nn.functional.gelu(x)
    if dist == "hot":                       # a tenth of the channels five times as large
        hot = torch.randperm(K, generator=gen, device="cuda")[:K // 10]
        x[:, hot] *= 5.0
    return x.to(dtype)


def _gradient(gen, M, N, dtype):
    return (torch.randn(M, N, generator=gen, device="cuda") * 1e-3).to(dtype)


def _set_layers(case):
    """(M, K, N, block, distribution) of every linear layer of the network."""
    rows, dim, b = case["batch"] * PATCHES, case["dim"], case["b"]
    one = [(case["batch"] * dim, PATCHES, PATCHES, 14, "normal"), (rows, dim, 4 * dim, b, "normal"),
           (rows, 4 * dim, dim, b, "gelu")]
    return one * case["layers"]


def _set_inputs(case, seed, gradients):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    dtype = DTYPES[case["dtype"]]
    out = []
    for M, K, N, b, dist in _set_layers(case):
        X = _activation(gen, M, K, dist, dtype)
        out.append((X, b, _gradient(gen, M, N, dtype) if gradients else None))
    return out


def _layer_inputs(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    dtype = DTYPES[case["dtype"]]
    X = _activation(gen, case["M"], case["K"], case["dist"], dtype)
    N = case["N"] if case["kind"] == "train" else case["K"]
    return X, _gradient(gen, case["M"], N, dtype)


def _blocks(M, K, br, bc):
    return -(-M // br), -(-K // bc)


class _Arena:
    """One buffer cut into pieces that start on 256-byte boundaries (how a program keeps what all layers save)."""

    def __init__(self, shapes, dtype):
        size = torch.empty((), dtype=dtype).element_size()
        at, places = 0, []
        for s in shapes:
            n = math.prod(s)
            places.append((at, n, s))
            at += -(-n * size // 256) * 256 // size
        self.buffer = torch.zeros(at, dtype=dtype, device="cuda")
        self.pieces = [self.buffer[a:a + n].view(s) for a, n, s in places]


def _set_arenas(inputs, keep):
    """mask, row_ptr, col_idx and values of every layer, and the kept blocks of each."""
    geo = [_blocks(X.shape[0], X.shape[1], b, b) for X, b, _ in inputs]
    kept = [B.bsr_keep_count(nbr * nbc, keep) for nbr, nbc in geo]
    mask = _Arena([(nbr * nbc,) for nbr, nbc in geo], torch.uint8)
    row_ptr = _Arena([(nbr + 1,) for nbr, _ in geo], torch.int32)
    col_idx = _Arena([(n,) for n in kept], torch.int32)
    values = _Arena([(n, b, b) for n, (_, b, _) in zip(kept, inputs)], inputs[0][0].dtype)
    return mask, row_ptr, col_idx, values, kept


def _ws(nbytes):
    return torch.empty(max(nbytes, 1), dtype=torch.uint8, device="cuda")


def prepare(case, seed):
    kind = case["kind"]
    if not kind.endswith("_set"):
        X, dY = _layer_inputs(case, seed)
        return dict(case=case, X=X, dY=dY)
    inputs = _set_inputs(case, seed, kind == "grad_set")
    mask, row_ptr, col_idx, values, kept = _set_arenas(inputs, case["keep"])
    bsr = list(zip(row_ptr.pieces, col_idx.pieces, values.pieces))
    select = B.SelectBatch([X for X, _, _ in inputs], [(b, b) for _, b, _ in inputs], [case["keep"]] * len(inputs),
                           mask.pieces)
    compress = B.CompressBatch([(X, b, b, m, n, *out) for (X, b, _), m, n, out in zip(inputs, mask.pieces, kept, bsr)])
    state = dict(case=case, select=select, select_ws=_ws(select.ws_bytes), compress=compress,
                 compress_ws=_ws(compress.ws_bytes))
    if kind == "prune_set":
        state["out"] = dict(mask=mask.buffer, row_ptr=row_ptr.buffer, col_idx=col_idx.buffer, values=values.buffer)
        return state
    # what the forward side of the step left behind
    _prune(state)
    state = dict(case=case)
    if kind == "restore_set":
        state["restore"] = B.DecompressBatch([(*out, X.shape[0], X.shape[1], b, b) for out, (X, b, _) in zip(bsr, inputs)])
    else:
        state["grad"] = B.MatmulBatch([(*out, X.shape[0], X.shape[1], b, b, dY) for out, (X, b, dY) in zip(bsr, inputs)])
        state["grad_ws"] = _ws(state["grad"].ws_bytes)
    return state


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------

def _prune(s):
    B.bsr_score_select_batched(s["select"], ws=s["select_ws"])
    B.bsr_compress_batched(s["compress"], ws=s["compress_ws"])


def run(state):
    c = state["case"]
    kind = c["kind"]
    if kind == "prune_set":
        _prune(state)
        return state["out"]
    if kind == "restore_set":
        return B.bsr_decompress_batched(state["restore"])
    if kind == "grad_set":
        return B.bsr_t_dense_matmul_batched(state["grad"], ws=state["grad_ws"])
    X, dY, M, K, br, bc = state["X"], state["dY"], c["M"], c["K"], c["br"], c["bc"]
    nbr, nbc = _blocks(M, K, br, bc)
    if kind == "sample":
        mask = B.bsr_score_select_grouped(X, br, bc, c["group_rows"], c["keep"])
        n_keep = B.bsr_grouped_keep_count(nbr, nbc, c["group_rows"], c["keep"])
        row_ptr, col_idx, values = B.bsr_compress(X, br, bc, mask, n_keep)
        grad = B.bsr_affine_scale_grad(row_ptr, col_idx, values, M, K, br, bc, dY)
    else:
        mask = B.bsr_score_select(X, br, bc, c["keep"])
        n_keep = B.bsr_keep_count(nbr * nbc, c["keep"])
        row_ptr, col_idx, values = B.bsr_compress(X, br, bc, mask, n_keep)
        grad = B.bsr_t_dense_matmul(row_ptr, col_idx, values, M, K, br, bc, dY)
    return dict(mask=mask, row_ptr=row_ptr, col_idx=col_idx, values=values, grad=grad)


def work(case):
    """Bytes that have to move (every input once, every output once) and the arithmetic on kept blocks."""
    kind, keep = case["kind"], case["keep"]
    e = 2 if case["dtype"] == "bf16" else 4
    if kind.endswith("_set"):
        layers = [(M, K, N, b, b) for M, K, N, b, _ in _set_layers(case)]
    else:
        layers = [(case["M"], case["K"], case.get("N", 0), case["br"], case["bc"])]
    nbytes = flops = 0.0
    for M, K, N, br, bc in layers:
        nbr, nbc = _blocks(M, K, br, bc)
        if kind == "sample":
            n_keep = B.bsr_grouped_keep_count(nbr, nbc, case["group_rows"], keep)
        else:
            n_keep = math.ceil(keep * (nbr * nbc))
        bsr = n_keep * (br * bc * e + 4) + 4 * (nbr + 1)
        if kind in ("train", "sample", "prune_set"):
            nbytes += M * K * e + nbr * nbc + bsr
            flops += 2.0 * M * K
        if kind == "restore_set":
            nbytes += bsr + M * K * e
        if kind == "grad_set":
            nbytes += bsr
        if kind in ("train", "grad_set"):
            nbytes += M * N * e + 4 * K * N
            flops += 2.0 * n_keep * br * bc * N
        if kind == "sample":
            nbytes += n_keep * br * bc * e + 4 * K          # of dY only what meets a kept block
            flops += 2.0 * n_keep * br * bc
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """Masks, indices and kept values are whole or copies; gradients are binary32 sums of up to M exact (bf16) or
    binary32 products, whose order an implementation is free to choose (at most 7e-7 from the 64-bit result, measured
    over all cases and some drawn ones)."""
    if case["kind"] in ("prune_set", "restore_set"):
        return "exact"
    return {"rel": 3e-6, "max": 3e-5}


# ---------------------------------------------------------------------------
# the same in 64 bits
# ---------------------------------------------------------------------------

def _padded(X, br, bc):
    """X as blocks [nbr, br, nbc, bc] in binary64, zeros beyond its edges."""
    (M, K), (nbr, nbc) = X.shape, _blocks(X.shape[0], X.shape[1], br, bc)
    P = torch.zeros(nbr * br, nbc * bc, dtype=torch.float64, device=X.device)
    P[:M, :K] = X
    return P.view(nbr, br, nbc, bc)


def _top(scores, n_keep):
    """The n_keep largest, the first of equals."""
    order = torch.sort(scores, descending=True, stable=True).indices[:n_keep]
    mask = torch.zeros(scores.numel(), dtype=torch.uint8, device=scores.device)
    mask[order] = 1
    return mask


def _exact_bsr(X, br, bc, keep, group_rows=None):
    P = _padded(X, br, bc)
    nbr, nbc = P.shape[0], P.shape[2]
    scores = P.square().sum(dim=(1, 3))
    step = group_rows or nbr
    mask = torch.cat([_top(s.reshape(-1), math.ceil(keep * s.numel())) for s in scores.split(step)]).view(nbr, nbc)
    row_ptr = torch.zeros(nbr + 1, dtype=torch.int64, device=X.device)
    row_ptr[1:] = mask.sum(1).cumsum(0)
    at = mask.nonzero()
    values = P.permute(0, 2, 1, 3)[at[:, 0], at[:, 1]]
    kept = mask.view(nbr, 1, nbc, 1) * P
    dense = kept.reshape(nbr * br, nbc * bc)[:X.shape[0], :X.shape[1]]
    return mask.view(-1), row_ptr.to(torch.int32), at[:, 1].to(torch.int32), values, dense


def exact(case, seed):
    kind = case["kind"]
    if not kind.endswith("_set"):
        X, dY = _layer_inputs(case, seed)
        mask, row_ptr, col_idx, values, dense = _exact_bsr(X, case["br"], case["bc"], case["keep"], case.get("group_rows"))
        if kind == "sample":
            grad = (dense * dY.double()).sum(0)
        else:
            grad = dense.t().contiguous() @ dY.double()
        return dict(mask=mask, row_ptr=row_ptr, col_idx=col_idx, values=values, grad=grad)
    inputs = _set_inputs(case, seed, kind == "grad_set")
    if kind == "grad_set":
        return [_exact_bsr(X, b, b, case["keep"])[4].t().contiguous() @ dY.double() for X, b, dY in inputs]
    if kind == "restore_set":
        return [_exact_bsr(X, b, b, case["keep"])[4] for X, b, _ in inputs]
    parts = [_exact_bsr(X, b, b, case["keep"])[:4] for X, b, _ in inputs]
    out = {}
    for k, (key, dtype) in enumerate((("mask", torch.uint8), ("row_ptr", torch.int32), ("col_idx", torch.int32),
                                      ("values", DTYPES[case["dtype"]]))):
        # laid out like the arena of the run: pieces on 256-byte boundaries of ITS element size
        size = torch.empty((), dtype=dtype).element_size()
        pieces = []
        for p in parts:
            v = p[k].reshape(-1)
            pad = -(-v.numel() * size // 256) * 256 // size - v.numel()
            pieces.append(torch.cat([v, torch.zeros(pad, dtype=v.dtype, device=v.device)]))
        out[key] = torch.cat(pieces)
    return out
