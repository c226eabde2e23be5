"""The hub tier (dense rows counted with matrix instructions over the heaviest
vertices) through the C ABI: whole results against the bitmap tier bit for
bit and sampled rows against the oracle, at the sizes where it can go wrong:
window and tile remainders, threshold sets of every register variant, rows of
255 and 256 members, groups with more members than have cursors, long lists
outside the hubs, row ranges and chunks."""
from __future__ import annotations

import numpy as np
import pytest

import hypergen as hg
import oracle

pytestmark = pytest.mark.gpu

WINDOW = 1 << 14


def hub_graph(m, hubs=60, p=0.3, extra=6, n=60_000, seed=1, wide=(), mid=0):
    """m rows: each hub with probability p, `extra` uniform vertices; rows in
    `wide` are filled up to the given size with further vertices; `mid`
    vertices outside the hubs lie in every 40th row (long lists)."""
    rng = np.random.default_rng(seed)
    rows, cols = np.nonzero(rng.random((m, hubs)) < p)
    r2 = np.repeat(np.arange(m), extra)
    c2 = rng.integers(hubs + mid, n, r2.size)
    r3 = np.repeat(np.arange(0, m, 40), mid)
    c3 = np.tile(np.arange(hubs, hubs + mid), len(range(0, m, 40)))
    key = np.unique(np.concatenate([rows, r2, r3]).astype(np.int64) * n + np.concatenate([cols, c2, c3]))
    parts = [key]
    for r, size in wide:
        have = key[key // n == r] % n
        free = np.setdiff1d(np.arange(hubs + mid, n), have)
        parts.append(r * n + rng.choice(free, size - have.size, replace=False))
    key = np.unique(np.concatenate(parts))
    he_ptr = np.concatenate([[0], np.cumsum(np.bincount(key // n, minlength=m))])
    return hg.from_csr(m, n, he_ptr, (key % n).astype(np.int32))


def check(inc, S, hub=True, seed=0):
    import torch
    import paper_2201_11326_amd as slg
    plain, ctx = slg.Context(0), slg.Context(0)
    plain.set_dense(0, 0)
    gp, g = plain.register_incidence(inc), ctx.register_incidence(inc)
    p = ctx.plan(g, S)
    st = p.stats()
    p.destroy()
    assert st["dense_slots"] > 0, st
    # only the hub tier keeps no survivors between the passes
    assert (st["dense_stored"] < st["dense_edges"]) == hub, st
    a, b = ctx.line_graph(g, S), plain.line_graph(gp, S)
    for x, y in zip(a, b):
        for f in ("row_ptr", "row", "col", "w"):
            assert torch.equal(getattr(x, f), getattr(y, f)), (x.s, f)
    rng = np.random.default_rng(seed)
    rows = np.unique(np.concatenate([[0, inc.m - 1], rng.integers(0, inc.m, 6)]))
    lg = a[0]
    ref = oracle.line_graph_rows(inc, lg.s, rows)
    rp = lg.row_ptr.cpu().numpy()
    for t, i in enumerate(ref.rows):
        rj, rw = ref.row(t)
        assert np.array_equal(lg.col[rp[i]:rp[i + 1]].cpu().numpy(), rj), int(i)
        assert np.array_equal(lg.w[rp[i]:rp[i + 1]].cpu().numpy(), rw), int(i)
    return ctx, g, a


# kept rows: just below, at and just above whole windows; thresholds of each
# register variant (1, 2, more), among them one that nothing reaches
@pytest.mark.parametrize("m, S", [(WINDOW + 1, [8]), (2 * WINDOW, [6, 9]), (2 * WINDOW + 1, [5, 7, 11]),
                                  (20_011, [7, 8, 9, 10, 12, 60]), (WINDOW + 511, [8, 70000])])
def test_hub_tier_equals_other_tiers_and_oracle(m, S):
    ctx, g, _ = check(hub_graph(m, seed=m), S, seed=m)
    g.release()
    ctx.close()


def test_row_sizes_at_the_tiers_bound():
    """255 members: the last size of the hub tier; 256: counted by the other
    tiers in the same plan."""
    inc = hub_graph(18_000, seed=3, wide=[(0, 255), (1, 256), (2, 254), (9_000, 257), (9_001, 255)])
    ctx, g, _ = check(inc, [8])
    g.release()
    ctx.close()


def test_largest_threshold_and_the_next():
    """s_min of 44 is the largest that the matrix operand's bias can hold."""
    inc = hub_graph(17_000, hubs=118, p=0.62, extra=2, seed=4)
    for s, hub in ((44, True), (45, False)):
        ctx, g, a = check(inc, [s], hub=hub)
        assert a[0].num_edges > 0
        g.release()
        ctx.close()


def test_members_beyond_the_cursors_and_long_lists():
    """Groups of rows with more than 32 members each outside the hubs are
    searched range by range; every 40th row shares 30 vertices outside the
    hubs, whose lists hold runs of equal steps."""
    ctx, g, _ = check(hub_graph(17_500, hubs=118, p=0.4, extra=70, n=200_000, seed=5, mid=9), [10, 20])
    g.release()
    ctx.close()


def test_stream_chunks_and_row_ranges():
    """Chunks cut hub rows anywhere; two row ranges reassemble the result."""
    import torch
    inc = hub_graph(2 * WINDOW + 77, seed=6)
    ctx, g, whole = check(inc, [8, 10])
    for rows in (None, ((0, 11_111), (11_111, inc.m))):
        got = {8: [], 10: []}

        def fn(k, s, r0, r1, e0, rp, ri, rj, rw):
            got[s].append((ri.clone(), rj.clone(), rw.clone()))

        for part in ([None] if rows is None else rows):
            ctx.line_graph_stream(g, [8, 10], 24 << 20, fn, rows=part)
        torch.cuda.synchronize()
        for lg in whole:
            assert len(got[lg.s]) > 2
            for t, f in enumerate(("row", "col", "w")):
                assert torch.equal(torch.cat([c[t] for c in got[lg.s]]), getattr(lg, f)), (lg.s, f)
    g.release()
    ctx.close()


@pytest.mark.parametrize("m, hubs, p, s, hub", [
    (20_000, 60, 0.2, 5, True),    # rows on both sides of two 2-paths per candidate
    (64_000, 100, 0.045, 3, False),  # 0.2 2-paths per pair of rows on average
])
def test_rows_and_graphs_below_the_tiers_ratio(m, hubs, p, s, hub):
    ctx, g, _ = check(hub_graph(m, hubs=hubs, p=p, extra=2, seed=m), [s], hub=hub)
    g.release()
    ctx.close()
