"""The work a program that serves a pruned model has this library do, as a list of timed cases: products with one
vector (lone launches, a decoder layer, batches of small matrices), with a few vectors at once, with FP16 and FP32
values, and the way from a dense pruned matrix to its first product.

Weights and vectors are drawn on the GPU from the seed alone: column keep-probabilities follow a Beta law (or are all the
same), part of the entries sits in planted dense blocks on scattered rows and columns, kept weights are N(0, 0.02^2), x is
N(0, 1): the recipe of workloads/generators.py, drawn in bulk.

A case is a dict:
  kind     "run"    one product through device.run
           "layer"  the seven products of a decoder layer, each in a launch of its own
           "groups" the same seven, one launch per group that is independent inside a layer (q+k+v, o, gate+up, down)
           "batch"  `count` matrices of one shape in one batched call
           "multi"  one matrix times `nb` vectors through device.run_multi
           "load"   build, upload and a first product, from the dense matrix in host memory
  m, n     shape ("layer" and "groups": n is the hidden size, m the size of the MLP)
  density, beta (0: every column alike), planted (share of the entries inside planted blocks)
  bits     width of a delta index; 0 leaves the library's default
  fp32     FP32 values, x and y instead of FP16
"""
import math

import numpy as np
import torch

import paper_2507_12205_amd as E
from paper_2507_12205_amd import device as D


def _case(name, kind, m, n, density, beta=2.0, planted=0.1, bits=4, fp32=False, nb=1, count=1):
    return dict(name=name, kind=kind, m=m, n=n, density=density, beta=beta, planted=planted, bits=bits, fp32=fp32, nb=nb,
                count=count)


def listed():
    return [
        # one projection of a 125M-parameter model at 50 % sparsity: the launch and the host's part are all there is
        _case("run 768x768 d4", "run", 768, 768, 0.5),
        # an attention projection of a 7B model, 50 % sparsity, every build option left at its default (8-bit deltas,
        # blocks of up to 8 rows)
        _case("run 4096x4096 default", "run", 4096, 4096, 0.5, bits=0),
        # odd sizes: rows that end inside a lane unit, an x that is no multiple of a vector load
        _case("run 2999x5003 d8", "run", 2999, 5003, 0.3, beta=0.5, planted=0.15, bits=8),
        # the second MLP matrix of a 13B model with a four times wider MLP, 80 % sparsity, unstructured: the widest x
        _case("run 5120x20480 d4", "run", 5120, 20480, 0.2, beta=0.0, planted=0.0),
        # one token through the projections of a 13B decoder layer at 70 % sparsity, a launch per projection
        _case("layer 5120/13824 d4", "layer", 13824, 5120, 0.3, beta=0.5, planted=0.15),
        # one token through the projections of a 7B decoder layer at 60 % sparsity, projections that read the same
        # activations sharing a launch
        _case("groups 4096/11008 d8", "groups", 11008, 4096, 0.4, bits=8),
        # twelve small projections that do not depend on one another in one call
        _case("batch 12x768x768 d4", "batch", 768, 768, 0.5, count=12),
        # two, four and eight sequences decoded together
        _case("multi 2x 4096x11008 d8", "multi", 4096, 11008, 0.4, bits=8, nb=2),
        _case("multi 4x 5120x13824 d4", "multi", 5120, 13824, 0.3, beta=0.5, planted=0.15, nb=4),
        _case("multi 8x 13824x5120 d4", "multi", 13824, 5120, 0.3, beta=0.5, planted=0.15, nb=8),
        # a model kept in FP32
        _case("run fp32 4096x11008 d8", "run", 4096, 11008, 0.4, bits=8, fp32=True),
        # loading: encode, upload and a first product of an attention projection
        _case("load 4096x4096 default", "load", 4096, 4096, 0.5, bits=0),
    ]


def _log_size(rng, lo, hi):
    v = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    # model sizes are mostly multiples of 64; every third size is left as it falls
    return v if rng.random() < 0.34 or v < 64 else v // 64 * 64


def draw(rng):
    kind = rng.choice(["run", "run", "run", "layer", "groups", "batch", "multi", "multi", "load"])
    density = round(rng.uniform(0.1, 0.5), 3)
    beta = rng.choice([0.0, 0.5, 2.0])
    planted = 0.0 if beta == 0.0 else rng.choice([0.1, 0.15])
    bits = rng.choice([0, 4, 4, 8])
    fp32 = rng.random() < 0.25
    nb = count = 1
    if kind in ("layer", "groups"):
        n = _log_size(rng, 512, 5120)
        m = int(n * rng.choice([2.6875, 2.7, 4.0]))
        if m * n > 13824 * 5120:
            m = 13824 * 5120 // n
        density = min(density, 0.3)
    elif kind == "batch":
        count = rng.randint(2, 16)
        m, n = _log_size(rng, 256, 2048), _log_size(rng, 256, 2048)
    elif kind == "load":
        m, n = _log_size(rng, 512, 4096), _log_size(rng, 512, 4096)
    else:
        m, n = _log_size(rng, 512, 20480), _log_size(rng, 512, 20480)
        if kind == "multi":
            nb = rng.choice([2, 4, 8])
            n = min(n, 8192 if fp32 else 16384)       # two vectors and their partial sums have to fit a compute unit's LDS
        while m * n * density > 20480 * 5120 * 0.2:
            m = max(256, m * 3 // 4)
            if m == 256:
                n = n * 3 // 4
    c = _case("", kind, m, n, density, beta, planted, bits, fp32, nb, count)
    del c["name"]
    return c


def _shapes(case):
    m, n = case["m"], case["n"]
    if case["kind"] in ("layer", "groups"):
        return [(n, n)] * 4 + [(m, n)] * 2 + [(n, m)]           # q, k, v, o, gate, up, down
    return [(m, n)] * case["count"]


def _weight(case, seed, k, m, n):
    """k-th dense pruned matrix of the case (on the GPU)."""
    g = torch.Generator(device="cuda").manual_seed(1000003 * seed + 17 * k + 1)
    rng = np.random.default_rng([seed, k, m, n])
    dt = torch.float32 if case["fp32"] else torch.float16
    blocks = int(case["planted"] * case["density"] * m * n / (16 * 32))
    background = case["density"] * (1.0 - case["planted"])
    if case["beta"] > 0:
        q = rng.beta(case["beta"], case["beta"], n)
        lo, hi = 0.0, 64.0
        for _ in range(40):                                     # scale so that the mean is the background density
            mid = 0.5 * (lo + hi)
            lo, hi = (mid, hi) if np.clip(mid * q, 0.02, 0.98).mean() < background else (lo, mid)
        p = np.clip(hi * q, 0.02, 0.98)
    else:
        p = np.full(n, background)
    keep = torch.rand((m, n), generator=g, device="cuda") < torch.from_numpy(p.astype(np.float32)).cuda()
    if blocks:
        rows = torch.randint(0, m, (blocks, 16, 1), generator=g, device="cuda")
        cols = torch.randint(0, n, (blocks, 1, 32), generator=g, device="cuda")
        keep.view(-1)[(rows * n + cols).view(-1)] = True
    w = torch.randn((m, n), generator=g, device="cuda").mul_(0.02).to(dt)
    return w.masked_fill_(~keep, 0)


def _vector(case, seed, k, n):
    g = torch.Generator(device="cuda").manual_seed(1000003 * seed + 17 * k + 2)
    dt = torch.float32 if case["fp32"] else torch.float16
    shape = (n, case["nb"]) if case["kind"] == "multi" else (n,)
    return torch.randn(shape, generator=g, device="cuda").to(dt)


def _inputs_of(case):
    """For every product of the pass, the index of the vector it reads."""
    if case["kind"] in ("layer", "groups"):
        return [0, 0, 0, 1, 2, 2, 3]        # q, k, v share one; o has its own; gate, up share one; down has its own
    return list(range(case["count"]))


def _build(case, w):
    opts = E.make_opts(delta_bits=case["bits"])
    return E.ecspmv_build_dense_f32(w, opts) if case["fp32"] else E.ecspmv_build_dense(w, opts)


def prepare(case, seed):
    shapes, which = _shapes(case), _inputs_of(case)
    dt = torch.float32 if case["fp32"] else torch.float16
    xs = {}
    for (m, n), v in zip(shapes, which):
        if v not in xs:
            xs[v] = _vector(case, seed, v, n)
    weights = [_weight(case, seed, k, m, n).cpu().numpy() for k, (m, n) in enumerate(shapes)]
    state = dict(case=case, kind=case["kind"], stream=int(torch.cuda.current_stream().cuda_stream))
    if case["kind"] == "load":
        state.update(w=weights[0], x=xs[0])
        return state
    mats = []
    for w in weights:
        a = _build(case, w)
        D.upload(a)
        mats.append(a)
    if case["kind"] == "multi":
        state.update(a=mats[0], x=xs[0], y=torch.empty((case["m"], case["nb"]), dtype=dt, device="cuda"))
        return state
    ys = [torch.empty(m, dtype=dt, device="cuda") for m, _ in shapes]
    state.update(ys=ys, xs=xs, mats=mats)
    if case["kind"] == "run":
        state.update(a=mats[0], x=xs[0], y=ys[0])
    elif case["kind"] == "layer":
        state["calls"] = [(a, xs[v].data_ptr(), y.data_ptr()) for a, v, y in zip(mats, which, ys)]
    else:
        groups = [(0, 1, 2), (3,), (4, 5), (6,)] if case["kind"] == "groups" else [tuple(range(case["count"]))]
        state["batches"] = [E.Batch([mats[i] for i in g], [xs[which[i]].data_ptr() for i in g], [ys[i].data_ptr() for i in g])
                            for g in groups]
    return state


def run(state):
    kind = state["kind"]
    if kind == "run":
        return D.run(state["a"], state["x"], state["y"])
    if kind == "multi":
        return D.run_multi(state["a"], state["x"], state["y"])
    if kind == "layer":
        for a, x, y in state["calls"]:
            a.ecspmv_run(x, y, state["stream"])
        return state["ys"]
    if kind == "load":
        case = state["case"]
        a = _build(case, state["w"])
        D.upload(a)
        y = torch.empty(case["m"], dtype=torch.float32 if case["fp32"] else torch.float16, device="cuda")
        return D.run(a, state["x"], y)
    for b in state["batches"]:
        b.ecspmv_run_batch(state["stream"])
    return state["ys"]


def work(case):
    """Every stored entry's value and delta once, every vector once, every result once (a load: the dense matrix once too)."""
    value = 4 if case["fp32"] else 2
    delta = (case["bits"] or 8) / 8
    shapes = _shapes(case)
    entries = sum(case["density"] * m * n for m, n in shapes)
    xs = {v: n for (_, n), v in zip(shapes, _inputs_of(case))}
    total = entries * (value + delta) + value * case["nb"] * (sum(xs.values()) + sum(m for m, _ in shapes))
    if case["kind"] == "load":
        total += value * case["m"] * case["n"]
    return {"bytes": total, "flops": 2.0 * entries * case["nb"]}


def tolerance(case):
    # FP16 results: the rounding of the result itself (2^-12 of it on average, 2^-11 at most; results far below the
    # typical one count against that) is all there is: two correct sums differ by at most one unit in the last place.
    # FP32 results: the order of the FP32 sums over up to some ten thousand entries.
    # Measured against the 64-bit results over the listed cases: 2.2e-4 and 1.1e-7; stated: about four times that.
    return {"rel": 5e-7, "max": 5e-6} if case["fp32"] else {"rel": 8e-4, "max": 2e-3}


def exact(case, seed):
    shapes, which = _shapes(case), _inputs_of(case)
    xs, ys = {}, []
    for k, ((m, n), v) in enumerate(zip(shapes, which)):
        if v not in xs:
            xs[v] = _vector(case, seed, v, n).double()
        w = _weight(case, seed, k, m, n)
        ys.append(torch.cat([w[r:r + 4096].double() @ xs[v] for r in range(0, m, 4096)]))
    return ys if case["kind"] in ("layer", "groups", "batch") else ys[0]
