"""sline_squeeze and sline_components on given pair lists, against the oracle:
one to three passes of the sort by second item, few and many pairs, fewer and
more pairs than items (components joins a sample first when there are more),
many components, one long row, and a squeeze without weights."""

from __future__ import annotations

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    from paper_2010_11448_amd import sline

    assert torch.cuda.is_available()
    c = sline.Context(0)
    yield c
    c.close()


def pairs(N: int, n: int, block: int, hub: bool, seed: int):
    """n pairs or fewer with both ends in the same block of ids, sorted; with
    `hub`, item N // 2 is in a pair with every third item."""
    rng = np.random.default_rng(seed)
    a = rng.integers(0, N, n)
    b = np.minimum(a - a % block + rng.integers(0, block, n), N - 1)
    if hub:
        x = np.arange(0, N, 3)
        a, b = np.concatenate([a, x]), np.concatenate([b, np.full(len(x), N // 2)])
    lo, hi = np.minimum(a, b), np.maximum(a, b)
    key = np.unique((lo * N + hi)[lo < hi])
    return (key // N).astype(np.int32), (key % N).astype(np.int32)


def chain(N: int, extra: int):
    a = np.arange(N - 1)
    lo = np.concatenate([a, np.zeros(extra, dtype=np.int64)])
    hi = np.concatenate([a + 1, 2 + np.arange(extra)])
    o = np.lexsort((hi, lo))
    return lo[o].astype(np.int32), hi[o].astype(np.int32)


CASES = [(2, 1, 2, False), (512, 5000, 512, True), (513, 5000, 7, True), (600, 200, 600, False),
         (600, 3000, 2, False), (5000, 400000, 5000, True), (262144, 300000, 300, True),
         (262145, 900000, 5, True), (300000, 1100000, 300000, False), (300000, 100000, 64, True)]


@pytest.mark.parametrize("case", CASES + [(1000, -1), (1000, 0), (1000, 1), (1000, 2), (70000, 64)],
                         ids=lambda c: "-".join(map(str, c)))
def test_pairs(ctx, case):
    import torch
    from paper_2010_11448_amd import sline

    N = case[0]
    if len(case) == 4:
        a, b = pairs(*case, seed=sum(case))
    else:  # a path with as many pairs as items less one, and `case[1]` more
        a, b = chain(N - 1 if case[1] < 0 else N, max(case[1], 0))
    w = np.random.default_rng(N).integers(-(1 << 30), 1 << 30, len(a)).astype(np.int32)
    print(f"case: {case} pairs={len(a)}", flush=True)
    ref = oracle.Pairs(a, b, w)
    L = sline.LineGraph(*[torch.from_numpy(x).cuda() for x in (a, b, w)])
    comp, count = ctx.components(L, N)
    want = oracle.components(N, ref)
    assert np.array_equal(comp.cpu().numpy(), want)
    present = np.zeros(N, dtype=bool)
    present[a] = present[b] = True
    assert count == int(np.sum(present & (want == np.arange(N))))
    old_id, Lq = oracle.squeeze(ref, N)
    rp, col, wq = oracle.adjacency(Lq, len(old_id))
    for flags in (0, sline.SLINE_NO_WEIGHTS):
        G = ctx.squeeze(L, N, flags)
        assert G["n_nodes"] == len(old_id) and G["n_arcs"] == 2 * len(a)
        assert np.array_equal(G["old_id"].cpu().numpy(), old_id)
        assert np.array_equal(G["row_ptr"].cpu().numpy(), rp)
        assert np.array_equal(G["col"].cpu().numpy(), col)
        if not flags:
            assert np.array_equal(G["w"].cpu().numpy(), wq)


def linked(N: int, *lists):
    lo = np.concatenate([np.minimum(x, y) for x, y in lists])
    hi = np.concatenate([np.maximum(x, y) for x, y in lists])
    key = np.unique((lo * N + hi)[lo < hi])
    return (key // N).astype(np.int32), (key % N).astype(np.int32)


def shapes(N: int):
    """Pairs whose ids follow their links, in one tree or several."""
    x = np.arange(N - 1)
    rng = np.random.default_rng(N)
    yield "path", linked(N, (x, x + 1))
    yield "two paths", linked(N, (x[:-1], x[:-1] + 2))
    yield "evens, then odds", linked(N, (x[:-1], x[:-1] + 2), (np.array([1]), np.array([(N - 1) // 2 * 2])))
    yield "there and back", linked(N, (x, N - 1 - x), (x, np.maximum(N - 2 - x, 0)))
    yield "paths of 100", linked(N, (x[x % 100 != 99], x[x % 100 != 99] + 1))
    yield "band", linked(N, *[(x[: N - k], x[: N - k] + k) for k in range(1, 20)])
    yield "grid", linked(N, (x, x + 1), (x[: N - 500], x[: N - 500] + 500))
    yield "tree", linked(N, ((x + 1) // 2, x + 1))
    yield "hub first", linked(N, (x * 0, x + 1))
    yield "hub last", linked(N, (x, x * 0 + N - 1))
    yield "hub between", linked(N, (x, x * 0 + N // 2))
    yield "two hubs", linked(N, (x[: N // 2], x[: N // 2] * 0 + 7), (x[N // 2 - 9 :], x[N // 2 - 9 :] * 0 + N - 1))
    p = rng.permutation(N)
    yield "path in any order", linked(N, (p[:-1], p[1:]))
    yield "half as many", linked(N, (rng.integers(0, N, N // 2), rng.integers(0, N, N // 2)))
    yield "twice as many", linked(N, (rng.integers(0, N, 2 * N), rng.integers(0, N, 2 * N)))


@pytest.mark.parametrize("N", [70, 2001, 300000])
def test_components_of_shapes(ctx, N):
    import torch
    from paper_2010_11448_amd import sline

    for name, (a, b) in shapes(N):
        print(f"case: {name}, {N} items, {len(a)} pairs", flush=True)
        w = np.ones(len(a), dtype=np.int32)
        want = oracle.components(N, oracle.Pairs(a, b, w))
        L = sline.LineGraph(*[torch.from_numpy(x).cuda() for x in (a, b, w)])
        for _ in range(3):
            comp, count = ctx.components(L, N)
            assert np.array_equal(comp.cpu().numpy(), want), name
            present = np.zeros(N, dtype=bool)
            present[a] = present[b] = True
            assert count == int(np.sum(present & (want == np.arange(N))))
