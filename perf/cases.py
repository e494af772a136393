"""The work that users of this library have it do, as a list of cases with a common interface:
training steps and inference of the model families over the range of graph sizes, layer widths,
storage types and arithmetics, single wide or very large layers, and the two preprocessing jobs
(building the normalised matrix from an edge list, and the reverse Cuthill-McKee reordering).

listed() names the cases, draw() gives further ones of the same ranges, prepare() makes what a
program holds before the call, run() is one pass through the public entry points, work() the
bytes and operations such a pass cannot do without, tolerance() how far two correct
implementations at the same precision may be apart.
"""
import math

import torch

import paper_2501_01951_amd as mg
from paper_2501_01951_amd.model import padded_rows

DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16}


# ---- cases --------------------------------------------------------------------------------------

def listed():
    return [
        # two-layer GCN on a 4096-node Erdos-Renyi graph (the smallest benchmark configuration):
        # a training step that is all launches and latency
        {"name": "gcn_step_4k_f32", "kind": "gcn", "graph": "uniform", "n": 4096, "degree": 10,
         "dims": "64-32-8", "dtype": "f32", "arith": "fp32"},
        # inference with a trained three-layer model on a small graph of odd size, bf16 storage
        {"name": "gcn_infer_20k_bf16", "kind": "infer", "graph": "rmat", "n": 19997, "degree": 16,
         "dims": "100-256-256-47", "dtype": "bf16", "arith": "fp32"},
        # the three-layer GCN of the R-MAT scale 20 configuration, one epoch, fp32
        {"name": "gcn_step_1m_f32", "kind": "gcn", "graph": "rmat", "n": 1 << 20, "degree": 32,
         "dims": "128-256-256-16", "dtype": "f32", "arith": "fp32"},
        # a dense social graph of the Reddit shape of the paper's Table 2 (233K nodes, 115M
        # entries, 602 features, 41 classes; 3 x 128 hidden), with the update products on the
        # bf16 matrix cores (three exact terms per fp32 operand)
        {"name": "gcn_step_233k_bf16x3", "kind": "gcn", "graph": "powerlaw", "n": 232965, "degree": 492,
         "dims": "602-128-128-41", "dtype": "f32", "arith": "bf16x3"},
        # the three-layer GCN of the 2.45M-node configuration, one epoch, bf16 storage
        {"name": "gcn_step_2m_bf16", "kind": "gcn", "graph": "rmat", "n": 2450000, "degree": 50,
         "dims": "100-256-256-47", "dtype": "bf16", "arith": "fp32"},
        # one wide layer (128 -> 1024, ReLU), forward and backward: the compute-bound shape
        {"name": "layer_2m_128_1024_f32", "kind": "layer", "graph": "rmat", "n": 1 << 21,
         "degree": 16, "dims": "128-1024", "dtype": "f32", "arith": "fp32", "relu": True},
        # one layer on a power-law graph too large for any cache (the largest configuration's
        # recipe at a tenth of its node count), forward and backward without ReLU
        {"name": "layer_11m_128_128_f32", "kind": "layer", "graph": "powerlaw", "n": 11100000,
         "degree": 29, "dims": "128-128", "dtype": "f32", "arith": "fp32", "relu": False},
        # GraphSAGE (mean aggregator, concatenation), one epoch
        {"name": "sage_step_1m_f32", "kind": "sage", "graph": "rmat", "n": 1 << 20, "degree": 32,
         "dims": "128-128-128-16", "dtype": "f32", "arith": "fp32"},
        # GIN (sum aggregator, two-layer perceptrons) on a medium graph of odd size, bf16 storage
        {"name": "gin_step_100k_bf16", "kind": "gin", "graph": "rmat", "n": 100003, "degree": 24,
         "dims": "128-128-128-16", "dtype": "bf16", "arith": "fp32"},
        # GCN with dropout on every aggregation (the masked product of Eq. 4), medium graph
        {"name": "dropout_step_262k_f32", "kind": "dropout", "graph": "rmat", "n": 1 << 18,
         "degree": 32, "dims": "128-256-256-16", "dtype": "f32", "arith": "fp32"},
        # preprocessing: normalised CSR from the edge list of the R-MAT scale 20 configuration
        {"name": "build_1m", "kind": "build", "graph": "rmat", "n": 1 << 20, "degree": 32},
        # preprocessing: reverse Cuthill-McKee positions of a three-dimensional grid whose ids
        # are scrambled (a mesh, the kind of graph that has a banded form)
        {"name": "rcm_grid_262k", "kind": "rcm", "graph": "grid", "n": 1 << 18, "degree": 6},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _width(rng, lo, hi):
    """A layer width: half of them round (a multiple of 32), half of them any number."""
    w = _log_int(rng, lo, hi)
    return max(32, (w + 16) // 32 * 32) if rng.random() < 0.5 else w


def _drawn(rng):
    kind = rng.choice(["gcn", "gcn", "gcn", "infer", "infer", "layer", "layer", "sage", "gin",
                       "dropout", "build", "rcm"])
    graph = rng.choice(["rmat", "rmat", "uniform", "powerlaw"])
    case = {"kind": kind, "graph": graph, "n": _log_int(rng, 2500, 2500000),
            "degree": _log_int(rng, 4, 100)}
    if kind == "build":
        case["n"] = _log_int(rng, 2500, 4000000)
        return case
    if kind == "rcm":
        case["graph"] = rng.choice(["grid", "rmat"])
        case["n"] = _log_int(rng, 2500, 500000)
        case["degree"] = 6 if case["graph"] == "grid" else case["degree"]
        return case
    if kind in ("gcn", "infer", "dropout"):
        hidden = _width(rng, 32, 256)
        dims = [_width(rng, 50, 602)] + [hidden] * rng.choice([1, 2, 2]) + [rng.randint(2, 64)]
        if kind == "dropout":
            dims[0] = min(dims[0], 256)
    elif kind in ("sage", "gin"):
        # widths of whole 16-byte groups: the concatenated halves of GraphSAGE need them
        dims = [8 * rng.randint(8, 32)] + [8 * rng.randint(8, 24)] * 2 + [8 * rng.randint(1, 6)]
    else:
        case["n"] = _log_int(rng, 20000, 8000000)
        dims = [_width(rng, 64, 256), _width(rng, 64, 1024)]
        case["relu"] = rng.random() < 0.5
    case["dims"] = "-".join(str(d) for d in dims)
    case["dtype"] = rng.choice(["f32", "f32", "bf16"])
    case["arith"] = "bf16x3" if case["dtype"] == "f32" and rng.random() < 0.25 else "fp32"
    return case


def _gathered(case):
    """Bytes of gathered feature rows and update operations of a pass, for keeping drawn cases
    below the largest listed one."""
    if "dims" not in case:
        return 0.0, 0.0
    dims = [int(d) for d in case["dims"].split("-")]
    e = 2 if case["dtype"] == "bf16" else 4
    entries = case["n"] * (case["degree"] + 1.0)
    passes = 1 if case["kind"] == "infer" else 2
    wide = 2.0 if case["kind"] in ("sage", "gin") else 1.0
    gathers = passes * entries * e * sum(dims[:-1])
    flops = 3.0 * passes * wide * case["n"] * sum(a * b for a, b in zip(dims, dims[1:]))
    return gathers, flops


def draw(rng):
    while True:
        case = _drawn(rng)
        gathers, flops = _gathered(case)
        entries = case["n"] * (case["degree"] + 1)
        most = {"build": 120e6, "rcm": 12e6}.get(case["kind"], 250e6)
        if entries <= most and gathers / 5.5e12 + flops / 8e13 <= 0.045 and \
                case["n"] * sum(int(d) for d in case.get("dims", "1").split("-")) <= 3e9:
            return case


# ---- inputs -------------------------------------------------------------------------------------

def _scramble(ids, n):
    """A fixed bijection of 0 .. n - 1, so that neighboring ids mean nothing."""
    mul = 0x9E3779B1 % n | 1
    while math.gcd(mul, n) != 1:
        mul += 2
    return (ids * mul + n // 3) % n


def _edges(case, gen):
    """Edge list (src, dst) of the case's graph as int32 device tensors; building with both
    directions of every edge gives about `degree` stored neighbors per node."""
    n, dev = case["n"], "cuda"
    count = n * case["degree"] // 2
    rand = lambda m: torch.rand(m, device=dev, generator=gen)
    if case["graph"] == "uniform":
        src = torch.randint(0, n, (count,), device=dev, generator=gen)
        dst = torch.randint(0, n, (count,), device=dev, generator=gen)
    elif case["graph"] == "rmat":
        # recursive matrix with quadrants (0.57, 0.19, 0.19, 0.05), squeezed onto n ids
        bits = max(1, (n - 1).bit_length())
        src = torch.zeros(count, dtype=torch.int64, device=dev)
        dst = torch.zeros(count, dtype=torch.int64, device=dev)
        for _ in range(bits):
            p = rand(count)
            down = p >= 0.76
            right = ((p >= 0.57) & (p < 0.76)) | (p >= 0.95)
            src.mul_(2).add_(down)
            dst.mul_(2).add_(right)
        src, dst = (src * n) >> bits, (dst * n) >> bits
        src, dst = _scramble(src, n), _scramble(dst, n)
    elif case["graph"] == "powerlaw":
        # source of rank r with probability ~ (r + r0)^(-1 / 1.1) (degree law with exponent 2.1,
        # largest expected degree at most 2^20), destination uniform
        beta, most = 1.0 / 1.1, min(1 << 20, max(2, n // 64))
        lo, hi = 1e-6, float(n)
        for _ in range(60):
            r0 = math.sqrt(lo * hi)
            top = count * (1 - beta) * r0 ** -beta / ((n + r0) ** (1 - beta) - r0 ** (1 - beta))
            lo, hi = (r0, hi) if top > most else (lo, r0)
        a, b = r0 ** (1 - beta), (n + r0) ** (1 - beta)
        rank = (a + rand(count).double() * (b - a)).pow_(1.0 / (1 - beta)).sub_(r0).long()
        src = _scramble(rank.clamp_(0, n - 1), n)
        dst = torch.randint(0, n, (count,), device=dev, generator=gen)
    else:
        # grid of about cubic shape over the first n cells, ids scrambled; a random twentieth of
        # the edges is missing, as in a mesh with holes
        side = max(2, round(n ** (1.0 / 3.0)))
        i = torch.arange(n, device=dev)
        ends = []
        for step, inside in ((1, i % side != side - 1), (side, i // side % side != side - 1),
                             (side * side, i >= 0)):
            u = i[inside & (i + step < n)]
            ends.append((u, u + step))
        src, dst = torch.cat([u for u, _ in ends]), torch.cat([v for _, v in ends])
        keep = rand(src.numel()) >= 0.05
        src, dst = _scramble(src[keep], n), _scramble(dst[keep], n)
    return src.to(torch.int32), dst.to(torch.int32)


def _weight(gen, rows, cols):
    """Glorot-uniform fp32 weights, rows padded to whole 16-byte groups."""
    a = math.sqrt(6.0 / (rows + cols))
    w = torch.empty(rows, (cols + 3) // 4 * 4, device="cuda")
    w.uniform_(-a, a, generator=gen)
    return w[:, :cols]


def _features(gen, n, f, dtype):
    t = padded_rows(n, f, dtype, "cuda")
    t.copy_(torch.randn(n, f, device="cuda", generator=gen))
    return t


class State:
    pass


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    s = State()
    s.case, s.n = case, case["n"]
    kind = case["kind"]
    if kind == "build":
        # one graph of this size, its nodes numbered and its edges ordered by the seed: the number
        # of stored entries, and with it the sizes of the results, is the same for every seed
        src, dst = _edges(case, torch.Generator(device="cuda").manual_seed(1))
        ids = torch.randperm(s.n, device="cuda", generator=gen).int()
        order = torch.randperm(src.numel(), device="cuda", generator=gen)
        s.src, s.dst = ids[src.long()[order]], ids[dst.long()[order]]
        return s
    src, dst = _edges(case, gen)
    flags = mg.SYMMETRIZE | (0 if kind == "sage" else mg.ADD_SELF_LOOPS)
    s.g = mg.build_csr(src, dst, s.n, flags)
    if kind == "rcm":
        return s
    if kind == "sage":
        mg.normalize(s.g, mg.NORM_MEAN)
    elif kind == "gin":
        mg.normalize(s.g, mg.NORM_SUM, eps=0.1)
    else:
        mg.normalize(s.g)
    del src, dst
    dims = [int(d) for d in case["dims"].split("-")]
    dt = DTYPES[case["dtype"]]
    L = len(dims) - 1
    s.arith = mg.ARITH_BF16X3 if case["arith"] == "bf16x3" else mg.ARITH_FP32
    x = _features(gen, s.n, dims[0], dt)
    if kind in ("infer", "layer"):
        s.pipe = mg.Pipeline()
    if kind == "layer":
        s.h = x
        s.w = _weight(gen, *dims)
        s.z = padded_rows(s.n, dims[0], dt, "cuda")
        s.out = padded_rows(s.n, dims[1], dt, "cuda")
        s.grad = _features(gen, s.n, dims[1], dt)
        s.dh = padded_rows(s.n, dims[0], dt, "cuda")
        s.dw = torch.empty_strided(s.w.shape, s.w.stride(), device="cuda")
        return s
    y = torch.randint(0, dims[-1], (s.n,), device="cuda", dtype=torch.int32, generator=gen)
    if kind == "sage":
        ws = [_weight(gen, 2 * dims[l], dims[l + 1]) for l in range(L)]
        s.step = mg.SAGEStep(s.g, x, ws, y)
    elif kind == "gin":
        w1 = [_weight(gen, dims[l], dims[l + 1]) for l in range(L)]
        w2 = [_weight(gen, dims[l + 1], dims[l + 1]) for l in range(L)]
        s.step = mg.GINStep(s.g, x, w1, w2, y)
    else:
        ws = [_weight(gen, dims[l], dims[l + 1]) for l in range(L)]
        if kind == "gcn":
            s.step = mg.GCNStep(s.g, x, ws, y)
        elif kind == "dropout":
            s.step = mg.GCNDropoutStep(s.g, x, ws, y, seed=seed, keep=0.5)
        else:
            s.w = ws
            s.order = [mg.UPDATE_FIRST if b < a else mg.AGG_FIRST for a, b in zip(dims, dims[1:])]
            s.z = [padded_rows(s.n, min(a, b), dt, "cuda") for a, b in zip(dims, dims[1:])]
            s.h = [x] + [padded_rows(s.n, d, dt, "cuda") for d in dims[1:]]
    return s


# ---- one pass -----------------------------------------------------------------------------------

def run(s):
    kind = s.case["kind"]
    if kind == "build":
        g = mg.build_csr(s.src, s.dst, s.n)
        mg.normalize(g)
        return g.arrays()  # copies: the graph's own arrays end with it
    if kind == "rcm":
        return mg.reorder_rcm(s.g)
    if s.arith != mg.ARITH_FP32:
        mg.set_update_arith(s.arith)
    try:
        if kind == "infer":
            L = len(s.w)
            for l in range(L):
                mg.layer_fwd(s.g, s.h[l], s.w[l], s.z[l], s.h[l + 1], s.pipe, relu=l < L - 1,
                             order=s.order[l])
            return s.h[L]
        if kind == "layer":
            relu = s.case["relu"]
            mg.layer_fwd(s.g, s.h, s.w, s.z, s.out, s.pipe, relu=relu)
            mg.layer_bwd(s.g, s.z, s.out, s.w, s.grad, s.dw, s.dh, s.pipe, relu=relu)
            return {"out": s.out, "dz": s.z, "dw": s.dw, "dh": s.dh}
        s.step.step()
    finally:
        if s.arith != mg.ARITH_FP32:
            mg.set_update_arith(mg.ARITH_FP32)
    t = s.step
    if kind == "gin":
        return {"logits": t.h[-1], "loss": t.loss, "dw1": t.dw1, "dw2": t.dw2}
    logits = t.logits if kind == "sage" else t.h[-1]
    return {"logits": logits, "loss": t.loss, "dw": t.dw}


# ---- what a pass cannot do without, and how exact it is -----------------------------------------

def work(case):
    n, kind = float(case["n"]), case["kind"]
    if case["graph"] == "grid":
        entries = n * 6.7  # 95 % of just under 3 n undirected edges, both directions, and loops
    else:
        entries = n * (case["degree"] + 1.0)
    matrix = 8.0 * entries + 8.0 * n  # columns and values once, row pointers once
    if kind == "build":
        # the edge list read, row pointers, columns, values, degrees and their roots written
        return {"bytes": 4.0 * n * case["degree"] + matrix + 8.0 * n, "flops": entries}
    if kind == "rcm":
        return {"bytes": 4.0 * entries + 12.0 * n, "flops": 0.0}
    dims = [int(d) for d in case["dims"].split("-")]
    e = 2.0 if case["dtype"] == "bf16" else 4.0
    L = len(dims) - 1
    train = kind != "infer"
    data_in = train and kind == "layer"  # the input gradient is wanted too
    bytes_, flops = 0.0, 0.0
    for l in range(L):
        a, b = dims[l], dims[l + 1]
        # Eq. 3 is associative: the aggregation runs at the narrower width where the model allows
        agg = float(min(a, b) if kind in ("gcn", "infer") else a)
        mul = float(a * b * (2 if kind == "sage" else 1) + (b * b if kind == "gin" else 0))
        down = l > 0 or data_in  # the gradient goes on to the layer below
        # forward: matrix and input read, output written
        bytes_ += matrix + e * n * (a + b)
        flops += 2.0 * entries * agg + 2.0 * n * mul
        if train:
            # weight gradient, and the gradient of the input through the transposed matrix;
            # activations and the gradient of the output read, the gradient of the input written
            narrow = kind == "gcn" and b < a
            agg_back = narrow or down
            bytes_ += e * n * (a + 2 * b) + 4.0 * mul
            flops += 2.0 * n * mul
            if agg_back:
                bytes_ += matrix
                flops += 2.0 * entries * agg
            if down:
                bytes_ += e * n * a
                flops += 2.0 * n * mul
    if train and kind != "layer":
        bytes_ += 2 * e * n * dims[-1] + 4.0 * n  # loss: logits and labels read, gradient written
    return {"bytes": bytes_, "flops": flops}


def tolerance(case):
    kind = case["kind"]
    if kind in ("build", "rcm"):
        # integers, and values that are defined by correctly rounded operations
        return "exact"
    if case["dtype"] == "bf16":
        # every stored tensor is rounded to 8 significant bits.  "max": a rounding, or a ReLU
        # derivative, that falls the other way upstream moves single elements by a few units
        return {"rel": 1e-2, "max": 0.9 if kind == "layer" and case["relu"] else 0.4}
    if kind == "infer" or (kind == "layer" and not case["relu"]):
        return {"rel": 2e-5}
    # The ReLU derivative of a pre-activation within rounding of zero can fall either way.  With
    # rounding errors of about 2e-7 of a pre-activation's size, a share of about 1e-7 of the
    # elements does, and a gradient with that share of its terms exchanged moves by the square root
    # of it in 2-norm: 3e-4, more on small tensors.  In a single layer's input gradient one such
    # element is a visible part of its row ("max").
    if kind == "layer":
        return {"rel": 1e-3, "max": 0.9}
    return {"rel": 1e-3}
