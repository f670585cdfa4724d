"""The counting kernels without hashed wedge lists, at the sizes where they turn:
the wedges and members a sieved item may have, more pairs than its table holds,
the widths of direct counters and of a range, tasks of several ranges, more
members than threads, and (s = 1) the pairs counted at a time."""

from __future__ import annotations

import numpy as np
import pytest

import oracle
from paper_2010_11448_amd import gen

from helpers import assert_same, to_device

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    from paper_2010_11448_amd import sline

    assert torch.cuda.is_available()
    c = sline.Context(0)
    yield c
    c.close()


def hub(T: int, k: int, r: int, N: int, seed: int) -> gen.Hypergraph:
    """Item 0 has k members; T of the N items after it, the last one among them,
    hold r of these (neighbours, cyclically) and all hold two vertices of their
    own, so nearly every item is kept up to s = 2.  Item 0 has r T wedges and T
    candidates that overlap it in r; members lie in about r T / k items."""
    st = gen.Stream(seed)
    at = np.sort(1 + np.argsort(st.uniform(N - 1), kind="stable")[:T - 1])
    at = np.append(at, N)
    first = st.integers(0, k - 1, T)
    shared = np.sort((first[:, None] + np.arange(r)) % k, axis=1)
    sizes = np.full(N + 1, 2, dtype=np.int64)
    sizes[0] = k
    sizes[at] += r
    rp = np.zeros(N + 2, dtype=np.int32)
    rp[1:] = np.cumsum(sizes)
    col = np.empty(rp[-1], dtype=np.int32)
    col[:k] = np.arange(k)
    end = rp[2:]
    col[end - 2] = k + 2 * np.arange(N)
    col[end - 1] = k + 2 * np.arange(N) + 1
    for q in range(r):
        col[rp[at] + q] = shared[:, q]
    return gen.Hypergraph(rp, col, N + 1, k + 2 * N)


CASES = [
    # sieved, one wave or four: wedges, members, pairs beyond the table
    (1024, 64, 2, 50000), (1025, 64, 2, 50000), (600, 65, 2, 50000), (1000, 8, 2, 9000),
    (4096, 256, 2, 70000), (4097, 256, 2, 70000), (1500, 257, 2, 70000), (4090, 40, 2, 200000),
    (700, 6, 5, 700), (2000, 12, 4, 2000),
    # direct counters of 4, 8 and 16 bits, one range and two
    (9000, 15, 3, 122880), (9000, 15, 3, 122882), (9000, 16, 3, 61440), (9000, 16, 3, 61442),
    (9000, 255, 3, 61442), (9000, 256, 3, 30720), (9000, 256, 3, 30722), (9000, 300, 3, 245800),
    # several tasks, more members than threads
    (45000, 90, 3, 400000), (30000, 1100, 4, 40000),
    # s = 1: wedges kept, a range and two, pairs counted at a time
    (8192, 30, 2, 9000), (8193, 30, 2, 9000), (3840, 30, 2, 245760), (3841, 30, 2, 245762),
]


@pytest.mark.parametrize("T,k,r,N", CASES, ids=["-".join(map(str, c)) for c in CASES])
def test_hub(ctx, T, k, r, N):
    import torch

    g = hub(T, k, r, N, seed=T + k + N)
    rp, col = to_device(g, torch.device("cuda", 0))
    base = ctx.tuning()
    for s in sorted({1, 2, r, r + 1}):
        ref, _ = oracle.wedge(g.row_ptr, g.col, g.n_edges, g.n_vertices, s, threads=8)
        for stage in (base["stage_max_bytes"], 0):
            what = f"T={T} k={k} r={r} N={N} s={s} stage={stage}"
            print(f"case: {what}", flush=True)
            ctx.set_tuning(stage_max_bytes=stage)
            try:
                assert_same(ctx.build(rp, col, g.n_vertices, s), ref, what)
            finally:
                ctx.set_tuning(**base)


def test_a_wedge_too_many_for_a_sieve(ctx):
    """8193 wedges in 17 ranges of 8-bit counters: one too many for the sieve and
    too few for direct counters, so the task kernel counts them, whatever its
    lookup-only members lower the planning cost to."""
    import torch

    T, k, r, N = 2731, 40, 3, 1000000
    g = hub(T, k, r, N, seed=5)
    rp, col = to_device(g, torch.device("cuda", 0))
    for s in (2, 3):
        ref, _ = oracle.wedge(g.row_ptr, g.col, g.n_edges, g.n_vertices, s, threads=8)
        print(f"case: {r * T} wedges N={N} s={s}", flush=True)
        assert_same(ctx.build(rp, col, g.n_vertices, s), ref, f"s={s}")


# members of item 0, one fewer than s, and items after it: counters of 4, 8 and 16
# bits that are all ones at s - 1, one range of them and two
UNPRUNED = [(15, 122878), (15, 122882), (255, 61438), (255, 61442), (65535, 30718), (65535, 30722)]


@pytest.mark.parametrize("k,N", UNPRUNED, ids=["-".join(map(str, c)) for c in UNPRUNED])
@pytest.mark.parametrize("variant", ["prune", "f2"])
def test_fewer_members_than_s(ctx, k, N, variant):
    """Without degree pruning an item of fewer than s members is counted as well,
    and is in no pair; two items after it make the only one."""
    import torch
    from paper_2010_11448_amd import sline

    s = k + 1
    flags = sline.SLINE_NO_PRUNE if variant == "prune" else sline.VARIANT_FLAGS[variant]
    g = hub(9000, k, 3, N, seed=k + N)
    extra = np.arange(g.n_vertices, g.n_vertices + s, dtype=np.int32)
    row_ptr = np.append(g.row_ptr, g.row_ptr[-1] + s * np.array([1, 2])).astype(np.int32)
    g = gen.Hypergraph(row_ptr, np.concatenate([g.col, extra, extra]), g.n_edges + 2, g.n_vertices + s)
    rp, col = to_device(g, torch.device("cuda", 0))
    ref, _ = oracle.wedge(g.row_ptr, g.col, g.n_edges, g.n_vertices, s, threads=8)
    assert len(ref.a) == 1
    for at in (s, s - 1, 3):
        ref, _ = oracle.wedge(g.row_ptr, g.col, g.n_edges, g.n_vertices, at, threads=8)
        print(f"case: {k} members N={N} s={at} flags={flags}", flush=True)
        assert_same(ctx.build(rp, col, g.n_vertices, at, 0, flags), ref, f"k={k} N={N} s={at}")


@pytest.mark.parametrize("s", [1, 2, 12])
@pytest.mark.parametrize("share", [4, 2, 1.25])
def test_some_tasks_counted_again(ctx, s, share):
    """A pool that holds a part of the pairs: the fill pass skips the tasks that
    were staged, one after the other, among those it counts again."""
    import torch

    g = gen.uniform_hypergraph(3000, 300, 55, 65, seed=7)
    rp, col = to_device(g, torch.device("cuda", 0))
    ref, _ = oracle.wedge(g.row_ptr, g.col, g.n_edges, g.n_vertices, s, threads=8)
    base = ctx.tuning()
    print(f"case: s={s}, pool for 1/{share} of {len(ref.a)} pairs", flush=True)
    ctx.set_tuning(stage_max_bytes=int(8 * len(ref.a) / share))
    try:
        for _ in range(3):
            assert_same(ctx.build(rp, col, g.n_vertices, s), ref, f"s={s} share={share}")
    finally:
        ctx.set_tuning(**base)


@pytest.mark.parametrize("small_max", [1, 20, 30])
@pytest.mark.parametrize("T", [7, 8, 12, 18, 19, 30])
def test_lowered_cost_of_a_few_wedges(ctx, T, small_max):
    """Hash tables alone: an item of a few wedges more than small_max_wedges is
    planned by what its lookup-only members leave, but a lane, which counts every
    wedge of an item and has room for 32, does not take it for that."""
    import torch

    g = hub(T, 5, 5, 40000, seed=T)
    rp, col = to_device(g, torch.device("cuda", 0))
    base = ctx.tuning()
    ctx.set_tuning(dense_min_wedges=0, small_max_wedges=small_max)
    try:
        for s in (2, 3, 4, 5):
            ref, _ = oracle.wedge(g.row_ptr, g.col, g.n_edges, g.n_vertices, s, threads=8)
            print(f"case: {5 * T} wedges, small_max={small_max} s={s}", flush=True)
            assert_same(ctx.build(rp, col, g.n_vertices, s), ref, f"T={T} s={s}")
    finally:
        ctx.set_tuning(**base)


@pytest.mark.parametrize("dual", [0, 1])
@pytest.mark.parametrize("rows", ["shuffled", "repeated"])
def test_rows_not_checked(ctx, rows, dual):
    """SLINE_SKIP_VALIDATE lets rows in that are out of order or list a member
    twice.  The pairs are unspecified then (rows of items out of order still
    count), but the call returns and the next one counts as ever."""
    import torch
    from paper_2010_11448_amd import sline

    g = hub(62000, 255, 4, 140000, seed=1)
    if dual:
        v, e = np.repeat(np.arange(g.n_edges), np.diff(g.row_ptr)), g.col
        o = np.lexsort((v, e))
        row_ptr = np.concatenate([[0], np.cumsum(np.bincount(e, minlength=g.n_vertices))])
        g = gen.Hypergraph(row_ptr.astype(np.int32), v[o].astype(np.int32), g.n_vertices, g.n_edges)
    rp, col = to_device(g, torch.device("cuda", 0))
    if rows == "shuffled":
        row = np.repeat(np.arange(g.n_edges), np.diff(g.row_ptr))
        o = np.lexsort((np.random.default_rng(2).random(len(row)), row))
        broken = torch.from_numpy(g.col[o]).to(rp.device)
    else:
        broken = col // 4 * 4
    for s in (2, 4):
        print(f"case: rows {rows}, dual={dual} s={s}", flush=True)
        L = ctx.build(rp, broken, g.n_vertices, s, dual, sline.SLINE_SKIP_VALIDATE)
        ref, _ = oracle.wedge(g.row_ptr, g.col, g.n_edges, g.n_vertices, s, dual=dual, threads=8)
        if rows == "shuffled" and not dual:
            assert_same(L, ref, f"shuffled s={s}")
        assert_same(ctx.build(rp, col, g.n_vertices, s, dual), ref, f"in order s={s}")


# Sieved or counted directly: as many ranges of direct counters as a sieved item may
# not have and one more, as few wedges for them as direct counters take and fewer
RANGES = [(1025, 64, 2, 122879), (1025, 64, 2, 122880), (511, 65, 2, 122879), (512, 65, 2, 122879),
          (4096, 255, 2, 122879), (2731, 15, 3, 245759), (2731, 15, 3, 245760), (4096, 256, 2, 61439),
          (4096, 256, 2, 61440)]


@pytest.mark.parametrize("T,k,r,N", RANGES, ids=["-".join(map(str, c)) for c in RANGES])
def test_sieved_or_direct(ctx, T, k, r, N):
    import torch

    g = hub(T, k, r, N, seed=T + k + N)
    rp, col = to_device(g, torch.device("cuda", 0))
    for s in sorted({2, r, r + 1}):
        ref, _ = oracle.wedge(g.row_ptr, g.col, g.n_edges, g.n_vertices, s, threads=8)
        print(f"case: T={T} k={k} r={r} N={N} s={s}", flush=True)
        assert_same(ctx.build(rp, col, g.n_vertices, s), ref, f"T={T} k={k} r={r} N={N} s={s}")


@pytest.mark.parametrize("order", [1, -1], ids=["ascending", "descending"])
def test_ids_in_order_of_size(ctx, order):
    """Hyperedges numbered by size: candidates crowd at one end of every range."""
    import torch

    st = gen.Stream(3)
    m, n = 30000, 60000
    size = np.sort(2 + np.minimum(300, (st.uniform(m) ** -0.8).astype(np.int64)))[::order]
    row = np.repeat(np.arange(m), size)
    v = (n * st.uniform(len(row)) ** 3).astype(np.int64)
    key = np.unique(row * n + v)
    row_ptr = np.concatenate([[0], np.cumsum(np.bincount(key // n, minlength=m))])
    g = gen.Hypergraph(row_ptr.astype(np.int32), (key % n).astype(np.int32), m, n)
    rp, col = to_device(g, torch.device("cuda", 0))
    for dual in (0, 1):
        for s in (2, 3, 5):
            ref, _ = oracle.wedge(g.row_ptr, g.col, m, n, s, dual=dual, threads=8)
            print(f"case: order={order} dual={dual} s={s} pairs={len(ref.a)}", flush=True)
            assert_same(ctx.build(rp, col, n, s, dual), ref, f"order={order} dual={dual} s={s}")


@pytest.mark.parametrize("n,at", [(128, 1), (300, 2), (820, 3), (40000, 1)])
def test_few_long_lists(ctx, n, at):
    """Member lists of a few hundred to many thousand items, among them those of
    hubs with neighbouring ids, in several ranges of direct counters."""
    import torch

    m = 140000
    st = gen.Stream(n)
    row = np.repeat(np.arange(m), 3)
    v = (n * st.uniform(len(row)) ** (4 if n > 1000 else 1)).astype(np.int64)
    row, v = np.append(row, np.full(40, at)), np.append(v, np.arange(40))  # a larger row
    key = np.unique(row * n + v)
    row_ptr = np.concatenate([[0], np.cumsum(np.bincount(key // n, minlength=m))])
    g = gen.Hypergraph(row_ptr.astype(np.int32), (key % n).astype(np.int32), m, n)
    rp, col = to_device(g, torch.device("cuda", 0))
    for s in (2, 3):
        ref, _ = oracle.wedge(g.row_ptr, g.col, m, n, s, threads=8)
        print(f"case: {n} members, s={s}, longest list {np.bincount(g.col).max()}, pairs={len(ref.a)}", flush=True)
        assert_same(ctx.build(rp, col, n, s), ref, f"n={n} s={s}")


def near(m: int, n: int, lo: int, hi: int, width: int, far: float, seed: int) -> gen.Hypergraph:
    """m rows of up to lo..hi members within `width` vertices of the row's own
    place among n, a share `far` of them anywhere."""
    st = gen.Stream(seed)
    size = st.integers(lo, hi, m)
    row = np.repeat(np.arange(m), size)
    k = len(row)
    v = (row * n // m + st.integers(0, width - 1, k)) % n
    v = np.where(st.uniform(k) < far, st.integers(0, n - 1, k), v)
    key = np.unique(row * n + v)
    row_ptr = np.concatenate([[0], np.cumsum(np.bincount(key // n, minlength=m))])
    return gen.Hypergraph(row_ptr.astype(np.int32), (key % n).astype(np.int32), m, n)


# rows and vertices, sizes, width, share anywhere: candidates that crowd in a small
# part of the range, all of them or most, for items of few and of many wedges
NEAR = [(30000, 6000, 5, 30, 400, 0.0), (30000, 6000, 5, 30, 400, 0.05), (60000, 120000, 5, 30, 400, 0.0),
        (60000, 120000, 5, 30, 400, 0.05), (40000, 8000, 30, 70, 200, 0.02), (20000, 2000, 2, 6, 40, 0.3)]


@pytest.mark.parametrize("case", NEAR, ids=["-".join(map(str, c)) for c in NEAR])
@pytest.mark.parametrize("dual", [0, 1])
def test_ids_of_neighbours_close(ctx, case, dual):
    import torch

    g = near(*case, seed=case[0] + dual)
    rp, col = to_device(g, torch.device("cuda", 0))
    base = ctx.tuning()
    for s in (1, 2, 4):
        ref, _ = oracle.wedge(g.row_ptr, g.col, g.n_edges, g.n_vertices, s, dual=dual, threads=8)
        for stage in (base["stage_max_bytes"], 0):
            print(f"case: {case} dual={dual} s={s} stage={stage} pairs={len(ref.a)}", flush=True)
            ctx.set_tuning(stage_max_bytes=stage)
            try:
                assert_same(ctx.build(rp, col, g.n_vertices, s, dual), ref, f"{case} dual={dual} s={s}")
            finally:
                ctx.set_tuning(**base)
