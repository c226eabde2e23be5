"""What the hub tier keeps: hub rows have no survivor store, so a few dense
rows beside them get a store of their own size."""
from __future__ import annotations

import numpy as np
import pytest

import hypergen as hg
from test_gpu_hub import WINDOW, check, hub_graph

pytestmark = pytest.mark.gpu

S_MIN = 20
CHUNK = 4 << 16  # bytes of the store that a workgroup may leave unused; two workgroups on each of 256 CUs


def peak(inc):
    import paper_2201_11326_amd as slg
    ctx = slg.Context(0)
    g = ctx.register_incidence(inc)
    p = ctx.plan(g, [S_MIN])
    st = p.stats()
    p.destroy()
    srv = ctx.server(workers=1, mem_budget_bytes=0)
    r = srv.wait(srv.submit(g, [S_MIN]), timeout_ms=60_000)
    assert r is not None and r.ok
    edges = r.outs[0].num_edges
    del r
    used = srv.stats()["bytes_peak"] - 12 * edges
    srv.close()
    g.release()
    ctx.close()
    return used, st


def test_dense_store_follows_the_dense_rows():
    args = dict(seed=8, hubs=60, p=0.5)
    m = 2 * WINDOW + 99
    hub, st = peak(hub_graph(m, **args))
    assert st["dense_edges"] > 0 and st["dense_stored"] == 0, st  # no row outside the hub tier
    inc = hub_graph(m, wide=[(0, 256), (1, 300)], **args)
    both, st = peak(inc)
    rows = 2 * 100 * m  # more than two wide rows' 2-paths
    room = 4 * rows // S_MIN + 512 * CHUNK + (16 << 20)
    assert 4 * st["dense_two_paths"] // S_MIN > 4 * room, st  # of the hub rows with them
    assert both - hub <= room, (hub, both)
    ctx, g, _ = check(inc, [S_MIN])
    g.release()
    ctx.close()


def test_streamed_blocks_estimate_the_store_by_dense_rows():
    """Every eighth row is too wide for the tier: 1.5e8 survivors to store,
    7e7 places. The blocks are cut so that none runs full; every edge is as
    unstreamed."""
    import torch
    import paper_2201_11326_amd as slg
    m, n, hubs, s = 4 * WINDOW + 200, 400_000, 60, 15
    rng = np.random.default_rng(9)
    rows, cols = np.nonzero(rng.random((m, hubs)) < 0.5)
    extra = np.where(np.arange(m) % 8 == 3, 260, 6)
    r2 = np.repeat(np.arange(m), extra)
    key = np.unique(np.concatenate([rows.astype(np.int64) * n + cols,
                                    r2.astype(np.int64) * n + rng.integers(hubs, n, r2.size)]))
    inc = hg.from_csr(m, n, np.concatenate([[0], np.cumsum(np.bincount(key // n, minlength=m))]),
                      (key % n).astype(np.int32))
    ctx = slg.Context(0)
    g = ctx.register_incidence(inc)
    whole = ctx.line_graph(g, [s])[0]
    p = ctx.plan(g, [s])
    st = p.stats()
    p.destroy()
    places = 2 * 512 * CHUNK // 4
    assert 2 * places < st["dense_stored"] < st["dense_edges"] // 2, st  # both tiers
    ctx.set_count_store(8 * places, 0)  # half of it holds 4-byte entries
    ctx.reset_timing()
    got = []
    ctx.line_graph_stream(g, [s], 1 << 30, lambda k, s, a, b, e, rp, ri, rj, rw: got.append(
        (ri.clone(), rj.clone(), rw.clone())) and False)
    torch.cuda.synchronize()
    work = ctx.work()
    assert work["blocks"] > 2 and work["dense_store_full_blocks"] == 0, work
    for t, f in enumerate(("row", "col", "w")):
        assert torch.equal(torch.cat([c[t] for c in got]), getattr(whole, f)), f
    g.release()
    ctx.close()
