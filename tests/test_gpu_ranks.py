"""Builds whose member lists hold candidate ranks instead of item ids, and the
sizes where that choice turns: 2^17 items, and three in four of them kept."""

from __future__ import annotations

import numpy as np
import pytest

import oracle
from paper_2010_11448_amd import gen

from helpers import assert_same, to_device

pytestmark = pytest.mark.gpu

RANK_MIN = 1 << 17


@pytest.fixture(scope="module")
def ctx():
    import torch
    from paper_2010_11448_amd import sline

    assert torch.cuda.is_available()
    c = sline.Context(0)
    yield c
    c.close()


def _thinned(items: int, kept: int, rest: int, seed: int) -> gen.Hypergraph:
    """`kept` hyperedges of 3..9 members at random ids, the others of `rest` members."""
    st = gen.Stream(seed)
    sizes = np.full(items, rest, dtype=np.int64)
    sizes[np.argsort(st.uniform(items), kind="stable")[:kept]] = st.integers(3, 9, kept)
    n = 9000
    rp, col = gen._draw_rows(st, sizes, n, None)
    return gen.Hypergraph(rp, col, items, n)


@pytest.mark.parametrize("items,kept,rest", [
    (RANK_MIN - 1, 40000, 1),               # too few items
    (RANK_MIN, RANK_MIN * 3 // 4, 1),       # exactly three in four kept
    (RANK_MIN, RANK_MIN * 3 // 4 + 1, 1),   # one more: ids
    (RANK_MIN + 77, 1, 1),                  # a single kept item
    (2 * RANK_MIN, 3000, 0),                # more items than incidences
])
def test_ranks(ctx, items, kept, rest):
    import torch
    from paper_2010_11448_amd import sline

    dev = torch.device("cuda", 0)
    g = _thinned(items, kept, rest, seed=items + kept)
    rp, col = to_device(g, dev)
    for s in (2, 3):
        print(f"case: {items} items, {kept} kept, s={s}", flush=True)
        ref, _ = oracle.wedge(g.row_ptr, g.col, g.n_edges, g.n_vertices, s, threads=8)
        assert_same(ctx.build(rp, col, g.n_vertices, s), ref, f"{items}/{kept} s={s}")
        # both passes of a build that cannot stage its pairs
        base = ctx.tuning()
        ctx.set_tuning(stage_max_bytes=0)
        try:
            assert_same(ctx.build(rp, col, g.n_vertices, s), ref, f"{items}/{kept} s={s} unstaged")
        finally:
            ctx.set_tuning(**base)
        cap = len(ref.a) + 1
        out = [torch.full((cap,), -7, dtype=torch.int32, device=dev) for _ in range(3)]
        st, k = ctx.build_noalloc(rp, col, g.n_vertices, s, 0, 0, *out)
        assert st == sline.SLINE_OK and k == len(ref.a)
        assert_same(sline.LineGraph(*[t[:k] for t in out]), ref, f"{items}/{kept} s={s} noalloc")
