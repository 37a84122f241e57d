"""Performance cases: the calls a program that uses this package makes, over the sizes it makes them at.

Kinds of case, each through the package's public entry points:

single   quantise, build and sample one distribution (``quantize``, ``build``,
         ``sample``), every call allocating its own results
serve    sample a forest that the program built once and keeps (``sample``)
map      a 2D map as a marginal over rows and one distribution per row: the
         whole chain (``quantize``, ``build_batched``, ``sample_2d``), or, with
         ``kept``, only ``sample_2d`` on a forest built once
batch    many uneven distributions through a ``BatchedPlan`` (quantise, build
         and sample with every buffer preallocated), enqueued or, with
         ``graph``, replayed as one captured graph
diff     positions and their adjoint through ``RTFSample``, with a ``DiffPlan``
         or, without one, allocating and checking as it goes
quality  the comparison of two mappings: alias tables built and sampled, and
         the same points through the inverse

Everything is drawn on the GPU from the seed; sizes depend on the case alone.
"""
import math

import numpy as np
import torch

import paper_1901_05423_amd as rtf
from paper_1901_05423_amd import workloads
from paper_1901_05423_amd.plan import BatchedPlan, DiffPlan

DEV = "cuda:0"


def listed():
    return [
        # The smallest use: a table of 1024 weights rebuilt and sampled 2^16
        # times, where launches and latency count (the 1024-entry workload).
        {"name": "single-1k", "kind": "single", "n": 1024, "ratio": 1.0, "weights": "uniform",
         "S": 1 << 16, "points": "random", "x": True},
        # An ordinary table of an odd size (a light list, a per-item table),
        # rebuilt for each of its odd-sized batches of samples.
        {"name": "single-100003", "kind": "single", "n": 100003, "ratio": 0.5, "weights": "zipf",
         "S": 1000003, "points": "random", "x": True},
        # The skewed workload of the benchmark: 2^20 weights of a permuted
        # Zipf law, one guide cell per weight, 2^26 uniforms.
        {"name": "single-zipf-2e20", "kind": "single", "n": 1 << 20, "ratio": 1.0,
         "weights": "zipf", "S": 1 << 26, "points": "random", "x": True},
        # The headline benchmark: 2^24 uniform weights, 2^26 uniforms.
        {"name": "single-uniform-2e24", "kind": "single", "n": 1 << 24, "ratio": 0.25,
         "weights": "uniform", "S": 1 << 26, "points": "random", "x": True},
        # A server that answers batches of index-only queries on one kept
        # table (an odd number of weights).
        {"name": "serve-index", "kind": "serve", "n": 3 * (1 << 20) + 5, "ratio": 0.25,
         "weights": "uniform", "S": 1 << 22, "points": "random", "x": False},
        # A small environment map rebuilt each frame: 300 x 500 pixels and a
        # hundred thousand stratified pairs.
        {"name": "map-300x500", "kind": "map", "rows": 300, "cols": 500, "ratio": 0.25,
         "S": 100000, "points": "strata", "x": True, "kept": False},
        # The 2D workload of the benchmark: 4096 x 4096 log-normal map with
        # hot spots, 2^27 pairs, from a forest built once.
        {"name": "map-4096x4096", "kind": "map", "rows": 4096, "cols": 4096, "ratio": 0.25,
         "S": 1 << 27, "points": "random", "x": True, "kept": True},
        # A small batch of uneven tables replayed as one graph, the way a
        # program removes launch latency.
        {"name": "batch-333-graph", "kind": "batch", "D": 333, "lo": 16, "hi": 2048,
         "ratio": 0.25, "per_1k": 1000, "tile": 1024, "collapsed": False, "graph": True, "x": True},
        # The batched workload of the benchmark: 10,000 uneven distributions
        # of uniform or Pareto weights, 64 samples per 1000 weights, with the
        # choices the tuner makes for it.
        {"name": "batch-10000", "kind": "batch", "D": 10000, "lo": 16, "hi": 65536,
         "ratio": 0.125, "per_1k": 64, "tile": 1024, "collapsed": False, "graph": False, "x": True},
        # The differentiable workload of the benchmark: 256 distributions of
        # 4096 softplus weights, 2^20 uniforms each, forward and adjoint.
        {"name": "diff-256x4096", "kind": "diff", "D": 256, "n": 4096, "ratio": 0.25,
         "per": 1 << 20, "plan": True, "collapsed": True},
        # The adjoint of one large distribution, 2^22 weights and 2^24
        # uniforms, through autograd without a plan.
        {"name": "diff-1x4194304", "kind": "diff", "D": 1, "n": 1 << 22, "ratio": 0.25,
         "per": 1 << 24, "plan": False, "collapsed": False},
        # The quality study on the benchmark's map: alias tables of every row
        # built and sampled, and the inverse, on 2^22 Hammersley points.
        {"name": "quality-4096x4096", "kind": "quality", "rows": 4096, "cols": 4096, "k": 22},
    ]


def _log(rng, lo, hi):
    """An integer spread over [lo, hi] by its logarithm (any residue)."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(("single", "single", "serve", "map", "batch", "diff", "diff", "quality"))
    if kind in ("single", "serve"):
        return {"kind": kind, "n": _log(rng, 256, 1 << 24), "ratio": rng.choice((0.25, 0.5, 1.0)),
                "weights": rng.choice(("uniform", "zipf", "pow20", "mod32_pow25")),
                "S": _log(rng, 1024, 1 << 26), "points": rng.choice(("random", "random", "strata")),
                "x": rng.choice((True, True, False))}
    if kind == "map":
        return {"kind": kind, "rows": _log(rng, 16, 4096), "cols": _log(rng, 16, 4096),
                "ratio": rng.choice((0.25, 0.5, 1.0)), "S": _log(rng, 4096, 1 << 26),
                "points": rng.choice(("random", "random", "strata")),
                "x": rng.choice((True, True, False)), "kept": rng.choice((True, False))}
    if kind == "batch":
        hi = _log(rng, 64, 65536)
        D = _log(rng, 2, min(10000, (1 << 29) // hi // 8))
        return {"kind": kind, "D": D, "lo": 16, "hi": hi, "ratio": rng.choice((0.125, 0.25, 1.0)),
                "per_1k": _log(rng, 64, 4000), "tile": rng.choice((1024, 2048)),
                "collapsed": rng.choice((False, True)), "graph": rng.choice((False, True)),
                "x": rng.choice((True, True, False))}
    if kind == "diff":
        n = _log(rng, 16, 1 << 22)
        D = _log(rng, 1, max(1, min(256, (1 << 22) // n)))
        plan = rng.choice((True, False))
        return {"kind": kind, "D": D, "n": n, "ratio": rng.choice((0.25, 1.0)),
                "per": _log(rng, 64, max(64, min(1 << 22, (1 << 27) // D))),
                "plan": plan, "collapsed": plan and rng.choice((False, True))}
    return {"kind": kind, "rows": _log(rng, 64, 4096), "cols": _log(rng, 64, 4096),
            "k": rng.randint(14, 24)}


# ---- inputs ------------------------------------------------------------------


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _bits(g, count):
    """`count` raw 64-bit uniforms (xi = u 2^-64), as int64 bit patterns."""
    a = torch.randint(0, 1 << 32, (count,), dtype=torch.int64, device=DEV, generator=g)
    b = torch.randint(0, 1 << 32, (count,), dtype=torch.int64, device=DEV, generator=g)
    return (a << 32) | b


def _uniforms(g, count, points):
    """Independent uniforms, or one in each of `count` equal strata in order."""
    u = _bits(g, count)
    if points == "strata":
        w = (1 << 63) // count * 2  # width of a stratum, rounded down
        off = ((u >> 32) & 0xFFFFFFFF) * (w >> 32) + ((u & 0xFFFFFFFF) * (w >> 32) >> 32)
        u = torch.arange(count, dtype=torch.int64, device=DEV) * w + off
    return u


def _weights(g, n, kind):
    if kind == "uniform":
        return 1.0 - torch.rand(n, device=DEV, generator=g)
    if kind == "zipf":
        w = torch.arange(1, n + 1, dtype=torch.float64, device=DEV) ** -1.1
        return w[torch.randperm(n, device=DEV, generator=g)].float()
    # the periodic and power densities of the load-count table, jittered
    w = torch.from_numpy(workloads.table1_weights(kind, n)).to(DEV)
    return w * (0.5 + torch.rand(n, device=DEV, generator=g))


def _map(g, rows, cols):
    """Log-normal map with eight Gaussian hot spots: the marginal, then the
    rows, one after another, and their offsets."""
    img = torch.exp(1.5 * torch.randn(rows, cols, device=DEV, generator=g, dtype=torch.float64))
    c = torch.rand(8, 2, device=DEV, generator=g, dtype=torch.float64)
    yy = torch.arange(rows, device=DEV, dtype=torch.float64) + 0.5
    xx = torch.arange(cols, device=DEV, dtype=torch.float64) + 0.5
    ey = torch.exp(-((yy[None] - c[:, :1] * rows) ** 2) / 18.0)
    ex = torch.exp(-((xx[None] - c[:, 1:] * cols) ** 2) / 18.0)
    img = (img + 1e4 * (ey.t() @ ex)).float()
    v = torch.cat([img.double().sum(1).float(), img.reshape(-1)])
    eo = torch.zeros(rows + 2, dtype=torch.int64, device=DEV)
    eo[1:] = rows + cols * torch.arange(rows + 1, device=DEV)
    return v, eo


def _sizes(case):
    """The batch's sizes, log-uniform in [lo, hi], and its samples per table."""
    r = np.random.default_rng(case["D"] * 1000003 + case["hi"])
    n = np.floor(np.exp(r.uniform(np.log(case["lo"]), np.log(case["hi"]), size=case["D"])))
    n = np.clip(n.astype(np.int64), case["lo"], case["hi"])
    return n, (case["per_1k"] * n + 999) // 1000


def _offsets(counts):
    o = np.zeros(len(counts) + 1, np.int64)
    o[1:] = np.cumsum(counts)
    return torch.from_numpy(o).to(DEV)


def _inputs(case, seed):
    """The tensors of a case, before any call: what `prepare` hands to the
    package and `exact` computes from."""
    g, kind, s = _gen(seed), case["kind"], {}
    if kind in ("single", "serve"):
        s["v"] = _weights(g, case["n"], case["weights"])
        s["u"] = _uniforms(g, case["S"], case["points"])
    elif kind == "map":
        s["v"], s["eo"] = _map(g, case["rows"], case["cols"])
        s["u"] = torch.stack([_uniforms(g, case["S"], case["points"]), _bits(g, case["S"])], 1)
    elif kind == "batch":
        n, per = _sizes(case)
        s["eo"], s["so"] = _offsets(n), _offsets(per)
        u = 1.0 - torch.rand(int(n.sum()), device=DEV, generator=g)
        coin = torch.rand(case["D"], device=DEV, generator=g) < 0.5
        coin = torch.repeat_interleave(coin, torch.from_numpy(n).to(DEV))
        s["v"] = torch.where(coin, u ** (-1.0 / 1.2), u)
        s["u"] = _bits(g, int(per.sum()))
    elif kind == "diff":
        D = case["D"]
        z = torch.randn(D * case["n"], device=DEV, generator=g)
        s["v"] = torch.nn.functional.softplus(z)
        s["eo"] = torch.arange(D + 1, dtype=torch.int64, device=DEV) * case["n"]
        s["so"] = torch.arange(D + 1, dtype=torch.int64, device=DEV) * case["per"]
        s["u"] = _bits(g, D * case["per"])
        s["gx"] = torch.randn(D * case["per"], device=DEV, generator=g, dtype=torch.float64)
    else:
        s["v"], s["eo"] = _map(g, case["rows"], case["cols"])
        s["u"] = torch.from_numpy(workloads.hammersley_u64(1 << case["k"]).view(np.int64)).to(DEV)
    return s


def _cells(n, ratio):
    return max(1, int(round(ratio * n)))


def prepare(case, seed):
    s, kind = _inputs(case, seed), case["kind"]
    s["case"] = case
    if kind == "serve":
        q, _ = rtf.quantize(s.pop("v"))
        s["f"] = rtf.build(q, _cells(case["n"], case["ratio"]))
    elif kind == "map":
        s["co"] = rtf.cells_like(s["eo"], case["ratio"])
        if case["kept"]:
            q, _ = rtf.quantize(s.pop("v"), s["eo"])
            s["f"] = rtf.build_batched(q, s["eo"], s["co"])
    elif kind == "quality":
        s["q"], _ = rtf.quantize(s.pop("v"), s["eo"])
        s["f"] = rtf.build_batched(s["q"], s["eo"], rtf.cells_like(s["eo"], 0.25))
    elif kind == "batch":
        co = rtf.cells_like(s["eo"], case["ratio"])
        s["plan"] = BatchedPlan(s["eo"], co, s["so"], s["v"].numel(), int(co[-1].item()),
                                s["u"].numel(), want_x=case["x"], collapsed=case["collapsed"],
                                tile=case["tile"])
        if case["graph"]:
            s["graph"] = s["plan"].capture(s["v"], s["u"])
    elif kind == "diff":
        s["v"].requires_grad_(True)
        if case["plan"]:
            co = rtf.cells_like(s["eo"], case["ratio"])
            s["plan"] = DiffPlan(s["eo"], co, s["so"], s["v"].numel(), int(co[-1].item()),
                                 s["u"].numel(), collapsed=case["collapsed"])
    return s


# ---- one pass ----------------------------------------------------------------


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "single":
        q, scale = rtf.quantize(s["v"])
        f = rtf.build(q, _cells(case["n"], case["ratio"]))
        idx, x = rtf.sample(f, s["u"], want_x=case["x"])
        return {"q": q.view(torch.int32), "scale": scale, "idx": idx, "x": x}
    if kind == "serve":
        idx, x = rtf.sample(s["f"], s["u"], want_x=case["x"])
        return {"idx": idx, "x": x}
    if kind == "map":
        f = s.get("f")
        if f is None:
            q, _ = rtf.quantize(s["v"], s["eo"])
            f = rtf.build_batched(q, s["eo"], s["co"])
        rc, xy = rtf.sample_2d(f, s["u"], want_xy=case["x"])
        return {"rc": rc, "xy": xy}
    if kind == "batch":
        p = s["plan"]
        if case["graph"]:
            s["graph"].replay()
        else:
            p.run(s["v"], s["u"])
        return {"q": p.q.view(torch.int32), "scale": p.scale, "idx": p.idx, "x": p.x}
    if kind == "diff":
        if case["plan"]:
            x = rtf.RTFSample.apply(s["v"], s["u"], s["plan"])
        else:
            x = rtf.RTFSample.apply(s["v"], s["u"], s["eo"], s["so"], case["ratio"])
        (grad,) = torch.autograd.grad(x, s["v"], s["gx"])
        return {"x": x.detach(), "grad": grad}
    t = rtf.alias_build(s["q"], s["eo"])
    alias = rtf.alias_sample_2d(t, s["u"])
    inverse, _ = rtf.sample_2d(s["f"], s["u"], want_xy=False)
    return {"alias": alias, "inverse": inverse}


def work(case):
    """Bytes read once and written once (weights 4, uniforms 8, indices 4,
    positions 8, a kept record's worth of keys 16 per sample read), and the
    integer and FP64 operations of the mapping (about 30 a sample)."""
    kind = case["kind"]
    pos = 8 if case.get("x", True) else 0
    if kind == "single":
        n, S = case["n"], case["S"]
        return {"bytes": 8 * n + S * (12 + pos), "flops": 10 * n + 30 * S}
    if kind == "serve":
        return {"bytes": 16 * min(case["n"], case["S"]) + case["S"] * (12 + pos),
                "flops": 30 * case["S"]}
    if kind == "map":
        n, S = case["rows"] * (case["cols"] + 1), case["S"]
        table = 16 * min(n, 2 * S) if case["kept"] else 4 * n
        return {"bytes": table + 2 * S * (12 + pos), "flops": 60 * S}
    if kind == "batch":
        n, per = _sizes(case)
        n, S = int(n.sum()), int(per.sum())
        return {"bytes": 8 * n + S * (12 + pos), "flops": 10 * n + 30 * S}
    if kind == "diff":
        n, S = case["D"] * case["n"], case["D"] * case["per"]
        return {"bytes": 8 * n + S * 24, "flops": 20 * n + 60 * S}
    n, S = case["rows"] * (case["cols"] + 1), 1 << case["k"]
    return {"bytes": 4 * n + 32 * S, "flops": 20 * n + 60 * S}


# ---- the same in 64 bits, by plain torch -------------------------------------

_LOW = 0xFFFFFFFF


def _mul128(a, b):
    """The high and low 64-bit words of the unsigned products of int64 bit
    patterns."""
    al, ah = a & _LOW, (a >> 32) & _LOW
    bl, bh = b & _LOW, (b >> 32) & _LOW
    p0, p1, p2 = al * bl, al * bh, ah * bl
    mid = ((p0 >> 32) & _LOW) + (p1 & _LOW) + (p2 & _LOW)
    hi = ah * bh + ((p1 >> 32) & _LOW) + ((p2 >> 32) & _LOW) + (mid >> 32)
    return hi, a * b


def _quantised(v, eo):
    """(q int64, scale float64 per distribution) of float32 weights."""
    n = eo[1:] - eo[:-1]
    mx = torch.segment_reduce(v.detach(), "max", lengths=n).double()
    scale = 4294967295.0 / mx
    q = torch.round(v.detach().double() * torch.repeat_interleave(scale, n))
    q = torch.where(v.detach() > 0, q.clamp(1.0, 4294967295.0), torch.zeros_like(q))
    return q.to(torch.int64), scale


def _sums(q):
    G = torch.zeros(q.numel() + 1, dtype=torch.int64, device=q.device)
    G[1:] = torch.cumsum(q, 0)
    return G


def _position(G, eo, d, u):
    """Global index, offset in the interval and position of the uniforms u of
    the distributions d."""
    e0, e1 = eo[d], eo[d + 1]
    W = G[e1] - G[e0]
    t, lo = _mul128(u, W)
    i = torch.searchsorted(G, G[e0] + t, right=True) - 1
    i = torch.minimum(i, e1 - 1)
    low = ((lo >> 32) & _LOW).double() * 2.0 ** -32 + (lo & _LOW).double() * 2.0 ** -64
    frac = ((G[e0] + t - G[i]).double() + low) / (G[i + 1] - G[i]).double()
    return i, frac, ((i - e0).double() + frac) / (e1 - e0).double()


_STEP = 1 << 24


def exact(case, seed):
    kind = case["kind"]
    if kind == "quality" or not case.get("x", True):
        return None
    s = _inputs(case, seed)
    u, S = s["u"], s["u"].shape[0]
    eo = s.get("eo")
    if eo is None:
        eo = torch.tensor([0, case["n"]], dtype=torch.int64, device=DEV)
    q, scale = _quantised(s["v"], eo)
    G = _sums(q)
    zero = torch.zeros(1, dtype=torch.int64, device=DEV)
    if kind == "map":
        xy = torch.empty(S, 2, dtype=torch.float64, device=DEV)
        for a in range(0, S, _STEP):
            b = min(S, a + _STEP)
            r, _, xy[a:b, 0] = _position(G, eo, zero, u[a:b, 0])
            xy[a:b, 1] = _position(G, eo, r + 1, u[a:b, 1])[2]
        return {"rc": None, "xy": xy}
    x = torch.empty(S, dtype=torch.float64, device=DEV)
    if kind == "diff":
        B, X, F = (torch.zeros(q.numel(), dtype=torch.float64, device=DEV) for _ in range(3))
    for a in range(0, S, _STEP):
        b = min(S, a + _STEP)
        d = zero
        if "so" in s:
            d = torch.searchsorted(s["so"], torch.arange(a, b, device=DEV), right=True) - 1
        i, frac, x[a:b] = _position(G, eo, d, u[a:b])
        if kind == "diff":
            c = s["gx"][a:b] * scale[d] / (case["n"] * q[i].double())
            xi = ((u[a:b] >> 32) & _LOW).double() * 2.0 ** -32 + (u[a:b] & _LOW).double() * 2.0 ** -64
            B.index_add_(0, i, c)
            X.index_add_(0, i, c * xi)
            F.index_add_(0, i, c * frac)
    if kind == "diff":
        B, X = B.view(case["D"], -1), X.view(case["D"], -1)
        after = torch.flip(torch.cumsum(torch.flip(B, [1]), 1), [1]) - B
        grad = X.sum(1, keepdim=True) - after - F.view(case["D"], -1)
        return {"x": x, "grad": grad.reshape(-1)}
    return {"q": None, "scale": scale, "idx": None, "x": x}
