"""The work this library is used for, as cases that can be timed and compared.

A case is a dict of plain values.  `path` says how a program uses the library:

  matvec   one call of rsr_matvec_ex on a handle (one vector, or a batch of them)
  linear   one call of an RsrLinear module on the activations of several tokens
  step     the matrix products of one token step through several layers, captured once in a
           HIP graph and replayed, as a decode loop does; every layer has weights of its own
  load     a new weight matrix becomes a handle, and its first product is taken

Shapes and value distributions are those of bench.py and rsr_inputs.py; draw() spreads the
same kinds of work over the sizes around them.
"""
import math

import torch

import paper_2603_27462_amd as rsr
from paper_2603_27462_amd.linear import RsrLinear

KINDS = {"binary": rsr.RSR_BINARY, "2pass": rsr.RSR_TERNARY_2PASS, "fused": rsr.RSR_TERNARY_FUSED,
         "dense": rsr.RSR_DENSE_TERNARY_P2}
DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16}

# "+" joins sibling layers (same input) that share one stacked handle, a space separates products
LAYERS_2B = "2560x2560+640x2560+640x2560 2560x2560 6912x2560+6912x2560 2560x6912"
LAYERS_8B = "14336x4096 4096x14336 4096x4096"


def listed():
    return [
        # the paper's kernel micro-benchmark: a small binary matrix, one float32 vector, called
        # from Python; nearly all latency
        dict(name="binary_1024", path="matvec", kind="binary", rows=1024, cols=1024, k=8, dtype="f32",
             batch=1, zeros=0.5),
        # its middle size, ternary in two binary passes
        dict(name="2pass_4096", path="matvec", kind="2pass", rows=4096, cols=4096, k=8, dtype="f32",
             batch=1, zeros=1 / 3),
        # a few vectors on a matrix that fits no tile: odd sizes, rows and vectors off every alignment
        dict(name="ragged_batch3", path="matvec", kind="2pass", rows=1001, cols=2999, k=5, dtype="f32",
             batch=3, zeros=1 / 3),
        # the headline product, 4096x14336 with one bf16 vector, weights streamed from memory: the
        # down projections of 16 decoder blocks one after the other
        dict(name="decode_down", path="step", kind="fused", layers="4096x14336", blocks=16, k=8,
             dtype="bf16", batch=1, zeros=0.35),
        # one token through the layers of a 2B-class model, block heights chosen by the library,
        # siblings stacked
        dict(name="decode_2b", path="step", kind="fused", layers=LAYERS_2B, blocks=6, k=0, dtype="bf16",
             batch=1, zeros=0.4),
        # four sequences at once through the layers of an 8B-class model
        dict(name="decode_8b_batch4", path="step", kind="fused", layers=LAYERS_8B, blocks=4, k=0,
             dtype="bf16", batch=4, zeros=0.35),
        # the prompt of a request through one layer: a gate projection, 512 tokens ...
        dict(name="prefill_512", path="linear", kind="fused", rows=6912, cols=2560, k=0, dtype="bf16",
             batch=512, zeros=0.4),
        # ... and a long prompt through the largest layer
        dict(name="prefill_2048", path="linear", kind="fused", rows=4096, cols=14336, k=8, dtype="bf16",
             batch=2048, zeros=0.35),
        # a retrieval table of a million items, one query and 64 queries in one call
        dict(name="retrieval_1", path="matvec", kind="binary", rows=1 << 20, cols=256, k=0, dtype="f32",
             batch=1, zeros=-1.0),
        dict(name="retrieval_64", path="matvec", kind="binary", rows=1 << 20, cols=256, k=8, dtype="f32",
             batch=64, zeros=-1.0),
        # the dense packed kind with a small float32 batch
        dict(name="dense_batch16", path="matvec", kind="dense", rows=14336, cols=4096, k=0, dtype="f32",
             batch=16, zeros=0.35),
        # loading a layer: preprocessing and the first product
        dict(name="load_4096", path="load", kind="fused", rows=4096, cols=4096, k=8, dtype="bf16", batch=1,
             zeros=1 / 3),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _height(rng, kind):
    if kind == "dense":
        return 0
    return rng.choice([0, 4, 5, 6, 7, 8] if kind == "fused" else [0, 4, 6, 8, 9, 10, 12])


def draw(rng):
    use = rng.choice(["single", "single", "batch", "tokens", "step", "step", "table", "load"])
    kind = rng.choice(["binary", "2pass", "fused", "fused", "dense"])
    dtype = rng.choice(["f32", "bf16"])
    zeros = round(rng.uniform(0.3, 0.5), 3)
    if use == "step":
        hidden, ffn = 32 * rng.randint(40, 128), 32 * rng.randint(80, 448)
        kv = 32 * rng.randint(8, 40)
        siblings = bool(rng.randint(0, 1))
        join = "+" if siblings else " "
        text = join.join("%dx%d" % (r, hidden) for r in (hidden, kv, kv))
        text += " %dx%d " % (hidden, hidden) + join.join(["%dx%d" % (ffn, hidden)] * 2) + " %dx%d" % (hidden, ffn)
        kind = rng.choice(["fused", "fused", "2pass", "dense"])
        return dict(path="step", kind=kind, layers=text, blocks=rng.randint(2, 6), k=_height(rng, kind),
                    dtype="bf16", batch=1 if siblings else rng.choice([1, 1, 2, 4, 8]), zeros=zeros)
    if use == "table":
        kind = rng.choice(["binary", "binary", "fused"])
        return dict(path="matvec", kind=kind, rows=_log_uniform(rng, 20000, 1 << 20), cols=rng.randint(48, 256),
                    k=_height(rng, kind), dtype=dtype, batch=rng.choice([1, 1, rng.randint(2, 64)]), zeros=-1.0)
    rows, cols = _log_uniform(rng, 500, 14336), _log_uniform(rng, 500, 14336)
    if rows * cols > 4096 * 14336:
        rows = 4096 * 14336 // cols
    k = _height(rng, kind)
    if use == "load":
        rows = min(rows, 4096 * 4096 // cols)
        return dict(path="load", kind=kind, rows=rows, cols=cols, k=k, dtype=dtype, batch=1, zeros=zeros)
    if use == "tokens":
        kind = rng.choice(["fused", "fused", "2pass"])
        batch = min(_log_uniform(rng, 32, 2048), max(32, 2048 * 4096 * 4096 // (rows * cols)))
        return dict(path="linear", kind=kind, rows=rows, cols=cols, k=_height(rng, kind), dtype=dtype,
                    batch=batch, zeros=zeros)
    batch = 1 if use == "single" else rng.randint(2, 32)
    return dict(path="matvec", kind=kind, rows=rows, cols=cols, k=k, dtype=dtype, batch=batch, zeros=zeros)


# ------------------------------------------------------------------------------ inputs
def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _matrix(g, kind, rows, cols, zeros):
    """int8 entries: P(0) = zeros, the others +1 (binary) or +1 and -1 alike; zeros < 0: every
    column has a density of its own, drawn from [0.05, 0.5]."""
    if zeros < 0:
        density = 0.05 + 0.45 * torch.rand(cols, generator=g, device="cuda")
    else:
        density = torch.full((cols,), 1.0 - zeros, device="cuda")
    M = torch.empty((rows, cols), dtype=torch.int8, device="cuda")
    for at in range(0, rows, 1 << 17):
        u = torch.rand((min(1 << 17, rows - at), cols), generator=g, device="cuda")
        part = (u < density).to(torch.int8)
        if kind != "binary":
            part -= 2 * (u < 0.5 * density).to(torch.int8)
        M[at:at + part.shape[0]] = part
    return M


def _vectors(g, cols, case):
    shape = (cols,) if case["batch"] == 1 else (case["batch"], cols)
    if case["zeros"] < 0:                       # a query against a table: non-negative features
        x = torch.rand(shape, generator=g, device="cuda")
    else:                                       # activations
        x = torch.randn(shape, generator=g, device="cuda")
    return x.to(DTYPES[case["dtype"]])


def _shapes(text):
    """[[(rows, cols), ...siblings], ...products]"""
    return [[tuple(int(n) for n in layer.split("x")) for layer in product.split("+")] for product in text.split()]


class _Step:
    """The products of one token step on fixed input buffers, captured in a graph."""

    def __init__(self, case, g):
        kind, k = KINDS[case["kind"]], case["k"]
        self.calls = []
        for _ in range(case["blocks"]):
            for siblings in _shapes(case["layers"]):
                Ms = [_matrix(g, case["kind"], r, c, case["zeros"]) for r, c in siblings]
                x = _vectors(g, siblings[0][1], case)
                h = rsr.rsr_preprocess(Ms[0], k, kind) if len(Ms) == 1 else rsr.rsr_preprocess_stacked(Ms, k, kind)
                self.calls.append((h, x, [0.02 + 0.01 * i for i in range(len(Ms))]))
        self.products()                          # first calls outside the capture
        torch.cuda.synchronize()
        self.graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(self.graph):
            self.outputs = self.products()

    def products(self):
        out = []
        for h, x, scales in self.calls:
            if len(scales) == 1:
                out.append(rsr.rsr_matvec_ex(h, x, scale=scales[0]))
            else:
                out.extend(rsr.rsr_matvec_stacked(h, x, scales))
        return out


def prepare(case, seed):
    g = _generator(seed)
    if case["path"] == "step":
        return {"path": "step", "step": _Step(case, g)}
    M = _matrix(g, case["kind"], case["rows"], case["cols"], case["zeros"])
    x = _vectors(g, case["cols"], case)
    kind, k = KINDS[case["kind"]], case["k"]
    if case["path"] == "load":
        return {"path": "load", "M": M, "k": k, "kind": kind, "x": x}
    if case["path"] == "linear":
        return {"path": "linear", "layer": RsrLinear(M, scale=0.02, k=k, kind=kind), "x": x.unsqueeze(0)}
    return {"path": "matvec", "handle": rsr.rsr_preprocess(M, k, kind), "x": x}


def run(state):
    path = state["path"]
    if path == "step":
        state["step"].graph.replay()
        return state["step"].outputs
    if path == "matvec":
        return rsr.rsr_matvec_ex(state["handle"], state["x"])
    if path == "linear":
        return state["layer"](state["x"])
    handle = rsr.rsr_preprocess(state["M"], state["k"], state["kind"])
    return rsr.rsr_matvec_ex(handle, state["x"])


def work(case):
    bits = 1.0 if case["kind"] == "binary" else math.log2(3.0)
    item = 4 if case["dtype"] == "f32" else 2
    batch = case["batch"]
    if case["path"] == "step":
        nbytes = flops = 0.0
        for siblings in _shapes(case["layers"]):
            nbytes += batch * siblings[0][1] * item
            for r, c in siblings:
                nbytes += r * c * bits / 8 + batch * r * 4
                flops += 2.0 * r * c * batch
        return {"bytes": case["blocks"] * nbytes, "flops": case["blocks"] * flops}
    rows, cols = case["rows"], case["cols"]
    nbytes = rows * cols * bits / 8 + batch * (cols * item + rows * 4)
    if case["path"] == "load":
        # the int8 matrix is read; what the handle keeps of it is at least its information content,
        # and for the kinds with a permutation also two bytes per column of every block
        nbytes += rows * cols
        if case["kind"] != "dense":
            passes = 2 if case["kind"] == "2pass" else 1
            nbytes += passes * 2.0 * cols * math.ceil(rows / (case["k"] or 8))
    return {"bytes": nbytes, "flops": 2.0 * rows * cols * batch}


def tolerance(case):
    # float32 sums in another order: against the same product in float64 the relative error is at
    # most 8.6e-7 and the largest error 8.1e-6 over these ranges (ternary tables of some fifty
    # columns, where sums cancel); four times that
    return {"rel": 4e-6, "max": 4e-5}
