"""Member lists of the kept items alone, rows walked by a lane, a group or a
wave, and the combined rows of a batch, against the oracle: row lengths around
the lane's and the group's limits, as many rows as the switch between the two,
incidences around the sort's tiles and a wave's share, few and many kept."""

from __future__ import annotations

import numpy as np
import pytest

import oracle
from paper_2010_11448_amd import gen

from helpers import assert_same, to_device

pytestmark = pytest.mark.gpu

LENGTHS = np.array([0, 1, 2, 3, 15, 16, 17, 18, 31, 32, 33, 64, 65])


@pytest.fixture(scope="module")
def ctx():
    import torch
    from paper_2010_11448_amd import sline

    assert torch.cuda.is_available()
    c = sline.Context(0)
    yield c
    c.close()


def rows(size, n: int, seed: int):
    """A hypergraph with rows of exactly the given lengths (n >= 80): members in
    even steps round [0, n), half of the rows from one of 64 places in steps
    of one, so that they overlap."""
    rng = np.random.default_rng(seed)
    m = len(size)
    narrow = rng.integers(0, 2, m) == 0
    at = np.where(narrow, rng.integers(0, 64, m) * max(1, n // 64) + rng.integers(0, 3, m), rng.integers(0, n, m))
    step = np.where(narrow, 1, rng.integers(1, max(2, n // 80), m))
    rp = np.concatenate([[0], np.cumsum(size)])
    row = np.repeat(np.arange(m), size)
    v = (at[row] + (np.arange(rp[-1]) - rp[row]) * step[row]) % n
    key = np.sort(row * n + v)
    return gen.Hypergraph(rp.astype(np.int32), (key % n).astype(np.int32), m, n)


def lengths(m: int, nnz: int, seed: int):
    """m lengths with a sum of about nnz: mostly 0..3, the others from LENGTHS."""
    rng = np.random.default_rng(seed)
    size = rng.choice(LENGTHS[:4], m)
    at = rng.choice(m, min(m, max(1, nnz // 100)), replace=False)
    size[at] = rng.choice(LENGTHS, len(at))
    return size


@pytest.mark.parametrize("m,n,nnz", [(131071, 300000, 200000), (131072, 300000, 200000),
                                     (140000, 5000, 90000), (3000, 1 << 18, 8192),
                                     (900, 513, 9000), (300000, 1 << 20, 540000)])
def test_build(ctx, m, n, nnz):
    import torch

    g = rows(lengths(m, nnz, m + n), n, seed=m)
    rp, col = to_device(g, torch.device("cuda", 0))
    for s in (1, 2, 16, 17):
        print(f"case: m={m} n={n} nnz={len(g.col)} s={s}", flush=True)
        for dual in (0, 1):
            ref, _ = oracle.wedge(g.row_ptr, g.col, g.n_edges, g.n_vertices, s, dual=dual, threads=8)
            assert_same(ctx.build(rp, col, g.n_vertices, s, dual), ref, f"m={m} s={s} dual={dual}")


@pytest.mark.parametrize("sizes", [(1023, 1, 1024, 0, 1025, 4096, 63, 64, 65), (0, 0, 5), (40000, 3, 40001),
                                   (1 << 18, 7, 0)], ids=lambda s: "-".join(map(str, s)))
def test_batch(ctx, sizes):
    import torch

    graphs = []
    for q, z in enumerate(sizes):
        size = lengths(max(1, z // 3), z, q)
        size = size[np.cumsum(size) <= z]  # then one entry a row, up to z
        size = np.concatenate([size, np.ones(z - int(size.sum()), dtype=size.dtype)])
        graphs.append(rows(size, max(80, z // 2), seed=z + q))
    dev = [(*to_device(g, torch.device("cuda", 0)), g.n_vertices) for g in graphs]
    for first in (0, 1):
        dual = [(q + first) % 2 for q in range(len(sizes))]
        s = [1 + (3 * q + first) % 5 for q in range(len(sizes))]
        print(f"case: batch {sizes} dual={dual} s={s}", flush=True)
        got = ctx.build_batch(dev, s, dual)
        for q, g in enumerate(graphs):
            ref, _ = oracle.wedge(g.row_ptr, g.col, g.n_edges, g.n_vertices, s[q], dual=dual[q], threads=8)
            assert_same(got[q], ref, f"graph {q}")


@pytest.mark.parametrize("k", [2, 64, 255, 256, 257, 2047, 2048, 2049, 3000])
def test_lookup_members(ctx, k):
    """Lookup-only members of an item that the hashed task kernel counts: as
    many members as a lane's registers hold, fewer and more."""
    import torch

    from test_gpu_direct import hub

    r = min(k, 12)
    g = hub(2000, k, r, 9000, seed=k)
    rp, col = to_device(g, torch.device("cuda", 0))
    base = ctx.tuning()
    ctx.set_tuning(dense_min_wedges=0)
    try:
        for s in sorted({2, 3, r, r + 1}):
            print(f"case: k={k} s={s}", flush=True)
            ref, _ = oracle.wedge(g.row_ptr, g.col, g.n_edges, g.n_vertices, s, threads=8)
            assert_same(ctx.build(rp, col, g.n_vertices, s), ref, f"k={k} s={s}")
    finally:
        ctx.set_tuning(**base)


def distinct_rows(size, n: int, seed: int):
    rng = np.random.default_rng(seed)
    row_ptr = np.concatenate([[0], np.cumsum(size)]).astype(np.int32)
    col = [np.sort(rng.choice(n, k, replace=False)) for k in size]
    return gen.Hypergraph(row_ptr, np.concatenate(col).astype(np.int32), len(size), n)


@pytest.mark.parametrize("sizes", ["one_length", "mixed"])
def test_batch_of_long_rows(ctx, sizes):
    """Dual graphs of rows around what a wave takes at once and of many more
    entries, in one batch and its plan; a bad member or a row out of order at
    the end of a long row is refused."""
    import torch
    from paper_2010_11448_amd import sline

    dev = torch.device("cuda", 0)
    if sizes == "one_length":
        graphs = [distinct_rows(np.full(40, k), 9000, k) for k in (255, 256, 257, 2000)]
    else:
        some = np.array([0, 1, 16, 17, 255, 256, 257, 300, 3000, 64])
        graphs = [distinct_rows(np.resize(np.roll(some, k), m), 50000, k) for k, m in ((0, 10), (3, 90), (7, 140))]
    duals, ss = [1] * len(graphs), [2] * len(graphs)
    dg = [to_device(g, dev) for g in graphs]
    batch = [(rp, col, g.n_vertices) for (rp, col), g in zip(dg, graphs)]
    refs = [oracle.wedge(g.row_ptr, g.col, g.n_edges, g.n_vertices, 2, dual=1, threads=8)[0] for g in graphs]
    print(f"case: batch of long rows, {sizes}", flush=True)
    for L, ref in zip(ctx.build_batch(batch, ss, duals), refs):
        assert_same(L, ref, "batch")
    plan = sline.BatchPlan(ctx, batch, ss, duals)
    try:
        for L, ref in zip(plan.run(), refs):
            assert_same(L, ref, "plan")
        g, (rp, col) = graphs[-1], dg[-1]
        end = int(g.row_ptr[np.argmax(np.diff(g.row_ptr)) + 1])  # of the longest row
        keep = int(col[end - 1])
        for bad in (g.n_vertices, -1, int(col[end - 2])):
            print(f"case: member {bad} at the end of a long row", flush=True)
            col[end - 1] = bad
            assert plan.run_raw() == sline.SLINE_EINVAL
            with pytest.raises(sline.SlineError):
                ctx.build_batch(batch, ss, duals)
        col[end - 1] = keep
        for L, ref in zip(plan.run(), refs):
            assert_same(L, ref, "plan, mended")
    finally:
        plan.close()
