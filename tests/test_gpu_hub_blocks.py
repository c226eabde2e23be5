"""The hub tier over the row blocks of a stream: blocks without hub rows
first, lists of hub rows built anew for every block, membership bits built
once; every edge against the unstreamed result."""
from __future__ import annotations

import numpy as np
import pytest

import hypergen as hg
from test_gpu_hub import WINDOW

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S", [[8], [8, 10]])
@pytest.mark.parametrize("free", [(0, 11_000), (13_000, 24_000)], ids=["free_rows_first", "free_rows_between"])
def test_blocks(S, free):
    import torch
    import paper_2201_11326_amd as slg
    m, n, hubs = 2 * WINDOW + 77, 60_000, 60
    rng = np.random.default_rng(free[0])
    member = rng.random((m, hubs)) < 0.3
    member[free[0]:free[1]] = False  # these rows share vertices with few others
    rows, cols = np.nonzero(member)
    r2 = np.repeat(np.arange(m), 9)
    key = np.unique(np.concatenate([rows.astype(np.int64) * n + cols,
                                    r2.astype(np.int64) * n + rng.integers(hubs, n, r2.size)]))
    inc = hg.from_csr(m, n, np.concatenate([[0], np.cumsum(np.bincount(key // n, minlength=m))]),
                      (key % n).astype(np.int32))
    ctx = slg.Context(0)
    g = ctx.register_incidence(inc)
    p = ctx.plan(g, S)
    st = p.stats()
    p.destroy()
    assert st["dense_stored"] < st["dense_edges"], st  # the hub tier is used
    whole = ctx.line_graph(g, S)
    ctx.set_count_store(2 << 20, 0)
    for rows in (None, (0, m - 9_000), (12_000, m)):
        ctx.reset_timing()
        got = {s: [] for s in S}
        ctx.line_graph_stream(g, S, 48 << 20, lambda k, s, a, b, e, rp, ri, rj, rw: got[s].append(
            (a, rp.clone(), ri.clone(), rj.clone(), rw.clone())) and False, rows=rows)
        torch.cuda.synchronize()
        assert ctx.work()["blocks"] > 4
        r0, r1 = rows or (0, m)
        for lg in whole:
            e0, e1 = int(lg.row_ptr[r0]), int(lg.row_ptr[r1])
            for t, f in enumerate(("row", "col", "w")):
                assert torch.equal(torch.cat([c[2 + t] for c in got[lg.s]]), getattr(lg, f)[e0:e1]), (lg.s, f, rows)
            at = 0
            for a, rp, _, rj, _ in got[lg.s]:
                k = rp.numel() - 1
                assert torch.equal(rp + (e0 + at), lg.row_ptr[a:a + k + 1]), (lg.s, rows, a)
                at += rj.numel()
    g.release()
    ctx.close()
