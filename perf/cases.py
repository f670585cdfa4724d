"""Performance cases of libsline: what a user's program calls, over the sizes it calls it with.

Inputs follow the input laws of ``paper_2010_11448_amd.gen`` (uniform,
power-law and lognormal-batch hypergraphs), drawn with torch on the GPU so
that a full-size graph takes milliseconds: members are drawn with
replacement and a row keeps its distinct ones.  A case fixes its graphs up to
their ids; the seed numbers their hyperedges and vertices, which sets every
row, every walk and every pair, but not how many pairs there are.

A case is a dict of plain values:

``path``   the entry point: ``build`` / ``noalloc`` (one graph), ``batch`` /
           ``plan`` / ``serve`` (many graphs), ``sweep`` (one graph, several s),
           ``after`` (components and adjacency of an L_s)
``law``    ``uniform``: sizes uniform on [2, 20], n = 2.5 m;
           ``powerlaw``: Zipf(2.2) sizes, Zipf(1.8) vertex popularity, n = 2 m;
           ``lognormal``: Zipf(2.2) sizes up to 2000, uniform members, n = 2 m
``m``      hyperedges (of the largest graph, where there are several)
``graphs`` number of graphs of a batch, plan or catalog
``s``, ``dual``, ``weights`` as in ``Context.build``
"""

from __future__ import annotations

import math
import time

import numpy as np
import torch

from paper_2010_11448_amd import sline

SWEEP_S = (2, 4, 8, 16)  # the thresholds above 1 of the power-law benchmark


def listed():
    return [
        # a small hypergraph into the caller's buffers, as in a tight loop that
        # may not allocate: all latency and launches
        dict(name="uniform_500_noalloc", path="noalloc", law="uniform", m=500, s=2, dual=0, weights=True),
        # the 2,000 x 5,000 benchmark graph by the ordinary call
        dict(name="uniform_2000", path="build", law="uniform", m=2000, s=3, dual=0, weights=True),
        # one graph of the batch law's median size, by itself, its line graph
        dict(name="lognormal_20k_s1", path="build", law="lognormal", m=20011, s=1, dual=0, weights=True),
        # the ordinary line graph (s = 1, pairs only) of a mid-size power-law graph
        dict(name="powerlaw_200k_s1_pairs", path="build", law="powerlaw", m=200003, s=1, dual=0, weights=False),
        # the full-size benchmark graph at a small threshold: the largest result
        dict(name="powerlaw_1m_s2", path="build", law="powerlaw", m=1000000, s=2, dual=0, weights=True),
        # and at a large one, where most pairs are dropped
        dict(name="powerlaw_1m_s8", path="build", law="powerlaw", m=1000000, s=8, dual=0, weights=True),
        # its dual side: vertices that share hyperedges
        dict(name="powerlaw_1m_dual_s8", path="build", law="powerlaw", m=1000000, s=8, dual=1, weights=True),
        # many graphs at once, each with its own s, results allocated per call
        dict(name="batch_128", path="batch", law="lognormal", m=200000, graphs=128, s=12, dual=0, weights=True),
        # the same kind of batch with both sides mixed, replayed from its plan
        dict(name="plan_128", path="plan", law="lognormal", m=200000, graphs=128, s=12, dual=1, weights=True),
        # a resident catalog answering a burst of queries, both sides, s on 1..16
        dict(name="serve_16x64", path="serve", law="lognormal", m=100000, graphs=16, s=16, dual=1, weights=True),
        # one graph over all thresholds of the study
        dict(name="sweep_300k", path="sweep", law="powerlaw", m=300000, s=2, dual=0, weights=True),
        # what follows L_s in the pipeline: components, squeezed ids, adjacency
        dict(name="after_200k_s2", path="after", law="powerlaw", m=200000, s=2, dual=0, weights=True),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("uniform", "lognormal", "powerlaw", "powerlaw", "batch", "plan", "serve", "sweep", "after"))
    dual = rng.randrange(2)
    if kind == "uniform":
        return dict(path=rng.choice(("build", "noalloc")), law="uniform", m=_log_uniform(rng, 200, 20000),
                    s=rng.randint(1, 8), dual=dual, weights=rng.random() < 0.8)
    if kind == "lognormal":
        return dict(path="build", law="lognormal", m=_log_uniform(rng, 1000, 200000), s=rng.randint(1, 12),
                    dual=dual, weights=rng.random() < 0.8)
    if kind == "powerlaw":
        m = _log_uniform(rng, 20000, 1000000)
        return dict(path="build", law="powerlaw", m=m, s=rng.randint(1 if m <= 250000 else 2, 16), dual=dual,
                    weights=rng.random() < 0.8)
    if kind in ("batch", "plan"):
        return dict(path=kind, law="lognormal", m=_log_uniform(rng, 5000, 200000), graphs=_log_uniform(rng, 8, 128),
                    s=rng.randint(2, 12), dual=dual, weights=True)
    if kind == "serve":
        return dict(path="serve", law="lognormal", m=_log_uniform(rng, 5000, 100000), graphs=rng.randint(4, 16),
                    s=16, dual=dual, weights=True)
    return dict(path=kind, law="powerlaw", m=_log_uniform(rng, 20000, 300000 if kind == "sweep" else 200000),
                s=rng.randint(2, 4), dual=dual, weights=True)


# ------------------------------------------------------------------ inputs

def _zipf(gen, alpha, lo, hi, size):
    """Truncated Zipf: P(k) proportional to k^-alpha on [lo, hi]."""
    pmf = torch.arange(lo, hi + 1, dtype=torch.float64, device="cuda") ** -alpha
    cdf = torch.cumsum(pmf, 0)
    u = torch.rand(size, dtype=torch.float64, device="cuda", generator=gen) * cdf[-1]
    return lo + torch.searchsorted(cdf, u, right=True).clamp_(max=hi - lo)


def _csr(row, v, m, n):
    """int32 CSR of the distinct (row, member) pairs, every row ascending."""
    key = torch.unique(row * n + v)
    ptr = torch.searchsorted(key, torch.arange(m + 1, device="cuda") * n)
    return ptr.to(torch.int32), (key % n).to(torch.int32)


def _generator(seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    return gen


def _graph(law, m, gen, ids):
    """(row_ptr, col, n_vertices) of one graph on the GPU: drawn from gen, numbered from ids."""
    if law == "uniform":
        n = max(20, 5 * m // 2)
        size = torch.randint(2, 21, (m,), device="cuda", generator=gen)
    else:
        n = 2 * m
        top = 2000 if law == "lognormal" else max(2, m // 100)
        size = _zipf(gen, 2.2, 2, min(n, top), m)
    row = torch.repeat_interleave(torch.arange(m, device="cuda"), size)
    if law == "powerlaw":
        weight = torch.cumsum(_zipf(gen, 1.8, 1, max(1, m // 10), n).double(), 0)
        u = torch.rand(row.numel(), dtype=torch.float64, device="cuda", generator=gen) * weight[-1]
        v = torch.searchsorted(weight, u, right=True).clamp_(max=n - 1)
    else:
        v = torch.randint(0, n, (row.numel(),), device="cuda", generator=gen)
    row = torch.randperm(m, device="cuda", generator=ids)[row]
    v = torch.randperm(n, device="cuda", generator=ids)[v]
    return (*_csr(row, v, m, n), n)


def _graphs(case, gen, ids):
    """The graphs of a batch or catalog: m_g lognormal around 20,000, clipped."""
    z = torch.randn(case["graphs"], dtype=torch.float64, device="cuda", generator=gen)
    sizes = (z * 1.2 + math.log(20000)).exp().round().clamp(1000, case["m"]).long().tolist()
    return [_graph(case["law"], mg, gen, ids) for mg in sizes]


def prepare(case, seed):
    gen, ids = _generator(case["m"]), _generator(seed)
    rng = np.random.default_rng(case["m"])
    state = dict(case, flags=0 if case["weights"] else sline.SLINE_NO_WEIGHTS)
    if "graphs" in case:
        G = case["graphs"]
        graphs = _graphs(case, gen, ids)
        sides = [int(x) for x in rng.integers(0, 2, G)] if case["dual"] else [0] * G
        if case["path"] == "serve":
            server = sline.Server(0, hbm_budget_bytes=4 << 30, max_batch=64, workers=2)
            ids = [server.register(*g) for g in graphs]
            state["queries"] = [(ids[int(rng.integers(0, G))], int(rng.integers(1, case["s"] + 1)),
                                 int(rng.integers(0, 2)) if case["dual"] else 0) for _ in range(64)]
            state["server"] = server
        else:
            state["ctx"] = sline.Context(0)
            state["batch"] = (graphs, [int(x) for x in rng.integers(1, case["s"] + 1, G)], sides)
            if case["path"] == "plan":
                state["plan"] = sline.BatchPlan(state["ctx"], *state["batch"])
        return state
    state["ctx"] = sline.Context(0)
    state["graph"] = _graph(case["law"], case["m"], gen, ids)
    rp, col, n = state["graph"]
    if case["path"] == "noalloc":
        # the caller's result buffers: each wedge makes at most one pair
        deg = torch.bincount(col.long(), minlength=n) if not case["dual"] else (rp[1:] - rp[:-1]).long()
        room = int((deg * (deg - 1) // 2).sum()) + 1
        state["out"] = [torch.empty(room, dtype=torch.int32, device="cuda") for _ in range(3 if case["weights"] else 2)]
    if case["path"] == "after":
        state["items"] = n if case["dual"] else case["m"]
        state["L"] = state["ctx"].build(rp, col, n, case["s"], case["dual"])
    return state


# -------------------------------------------------------------------- runs

def _join(results):
    """The results of many graphs as one edge list each of a, b, w, and the pairs per graph."""
    return (torch.cat([L.a for L in results]), torch.cat([L.b for L in results]),
            torch.cat([L.w for L in results]), np.array([len(L) for L in results], dtype=np.int64))


def run(state):
    path = state["path"]
    if path == "build":
        L = state["ctx"].build(*state["graph"], state["s"], state["dual"], state["flags"])
        return L.a, L.b, L.w
    if path == "noalloc":
        a, b, *w = state["out"]
        status, n = state["ctx"].build_noalloc(*state["graph"], state["s"], state["dual"], state["flags"],
                                               a=a, b=b, w=w[0] if w else None)
        if status != sline.SLINE_OK:
            raise sline.SlineError(status, "build_noalloc")
        return [t[:n] for t in state["out"]]
    if path == "batch":
        graphs, s, sides = state["batch"]
        return _join(state["ctx"].build_batch(graphs, s, sides))
    if path == "plan":
        return _join(state["plan"].run())
    if path == "serve":
        server = state["server"]
        tickets = [server.submit(*q) for q in state["queries"]]
        results = []
        for t in tickets:
            while (got := server.poll(t)) is None:
                time.sleep(20e-6)
            results.append(got[0])
        return _join(results)
    if path == "sweep":
        s = [x for x in SWEEP_S if x >= state["s"]]
        return [(L.a, L.b, L.w) for L in state["ctx"].build_sweep(*state["graph"], s, state["dual"])]
    comp, count = state["ctx"].components(state["L"], state["items"])
    g = state["ctx"].squeeze(state["L"], state["items"])
    return comp, count, g["n_nodes"], g["old_id"], g["row_ptr"], g["col"], g["w"]


# -------------------------------------------------------------------- work

def _leaves(v):
    if isinstance(v, (list, tuple)):
        for x in v:
            yield from _leaves(x)
    elif v is not None:
        yield v


def work(case):
    """Input and output read and written once; one count per wedge (two items
    that share a member, items smaller than s left out)."""
    state = prepare(case, 0)
    out = sum(v.numel() * v.element_size() for v in _leaves(run(state)) if isinstance(v, torch.Tensor))
    if case["path"] == "after":
        L = state["L"]
        return {"bytes": 12 * len(L) + out, "flops": len(L)}
    if case["path"] == "serve":
        graphs = state["server"]._keep
        return {"bytes": out + sum(4 * (rp.numel() + col.numel()) for rp, col in
                                   (graphs[g] for g, _, _ in state["queries"])), "flops": out // 12}
    many = zip(*state["batch"]) if "batch" in state else [(state["graph"], case["s"], case["dual"])]
    read = wedges = 0
    for (rp, col, n), s, dual in many:
        read += 4 * (rp.numel() + col.numel())
        size = (rp[1:] - rp[:-1]).long()
        if dual:
            deg = torch.bincount(col.long(), minlength=n)
            kept = (deg >= s)[col.long()].long()
            d = torch.zeros_like(size).index_add_(0, torch.repeat_interleave(
                torch.arange(size.numel(), device="cuda"), size), kept)
        else:
            kept = torch.repeat_interleave(size >= s, size)
            d = torch.bincount(col.long()[kept], minlength=n)
        wedges += int((d * (d - 1) // 2).sum())
    return {"bytes": read + out, "flops": wedges}


def exact(case, seed):
    """For one small graph: the dense incidence product in 64 bits."""
    if case["path"] not in ("build", "noalloc") or case["law"] != "uniform" or case["m"] > 4000:
        return None
    rp, col, n = _graph(case["law"], case["m"], _generator(case["m"]), _generator(seed))
    rp, col = rp.cpu().numpy(), col.cpu().numpy()
    B = np.zeros((case["m"], n))
    B[np.repeat(np.arange(case["m"]), np.diff(rp)), col] = 1.0
    overlap = np.triu(B.T @ B if case["dual"] else B @ B.T, 1)
    a, b = np.nonzero(overlap >= case["s"])
    out = [a.astype(np.int32), b.astype(np.int32)]
    return out + [overlap[a, b].astype(np.int32)] if case["weights"] else out
