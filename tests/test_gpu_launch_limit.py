"""Launches that are split where the device takes no larger ones, with the
limit lowered so that small inputs take many: results equal those of single
launches and of the other tiers."""
from __future__ import annotations

import pytest

from test_gpu_hub import WINDOW, hub_graph

pytestmark = pytest.mark.gpu


def equal(a, b):
    import torch
    for x, y in zip(a, b):
        for f in ("row_ptr", "row", "col", "w"):
            assert torch.equal(getattr(x, f), getattr(y, f)), (x.s, f)


@pytest.mark.parametrize("limit", [7, 1000])
@pytest.mark.parametrize("S", [[8], [6, 9], [6, 8, 11]])
def test_hub_tier_in_many_launches(limit, S):
    import paper_2201_11326_amd as slg
    inc = hub_graph(2 * WINDOW + 77 if limit > 7 else WINDOW + 77, seed=limit)
    ctx, plain = slg.Context(0), slg.Context(0)
    plain.set_dense(0, 0)
    g, gp = ctx.register_incidence(inc), plain.register_incidence(inc)
    ctx.set_launch_limit(limit)
    with pytest.raises(slg.SlgError):
        ctx.set_launch_limit(-1)
    p = ctx.plan(g, S)
    assert p.stats()["dense_slots"] > 0
    p.destroy()
    equal(ctx.line_graph(g, S), plain.line_graph(gp, S))
    for x, h in ((ctx, g), (plain, gp)):
        h.release()
        x.close()


def test_late_row_ranges():
    """A streamed range's hub rows have slots from its own windows on."""
    import torch
    import paper_2201_11326_amd as slg
    inc = hub_graph(4 * WINDOW + 99, seed=3)
    ctx = slg.Context(0)
    g = ctx.register_incidence(inc)
    whole = ctx.line_graph(g, [9])[0]
    ctx.set_launch_limit(500)
    got = []
    cuts = [0, 64, WINDOW - 1, WINDOW, 2 * WINDOW + 63, 3 * WINDOW + 64, inc.m - 5, inc.m]
    for r0, r1 in zip(cuts, cuts[1:]):
        ctx.line_graph_stream(g, [9], 64 << 20, lambda k, s, a, b, e, rp, ri, rj, rw: got.append(
            (ri.clone(), rj.clone(), rw.clone())) and False, rows=(r0, r1))
    torch.cuda.synchronize()
    for t, f in enumerate(("row", "col", "w")):
        assert torch.equal(torch.cat([c[t] for c in got]), getattr(whole, f)), f
    g.release()
    ctx.close()


@pytest.mark.parametrize("store", [True, False])
@pytest.mark.parametrize("limit", [1, 2, 5, 33])
def test_light_classes_in_many_launches(limit, store):
    """Rows of every light class, against the oracle."""
    import numpy as np
    import hypergen as hg
    import oracle
    import paper_2201_11326_amd as slg
    ptr, idx, at = [0], [], 0
    for width, rows in ((3, 700), (5, 9), (12, 30), (17, 45), (24, 50), (33, 70), (46, 95)):
        for r in range(rows):  # row r of a band shares width - d vertices with row r + d
            idx.extend(range(at + r, at + r + width))
            ptr.append(len(idx))
        at += rows + width
    inc = hg.from_csr(len(ptr) - 1, at, np.array(ptr, np.int64), np.array(idx, np.int32))
    ctx = slg.Context(0)
    if not store:
        ctx.set_count_store(0)
    ctx.set_launch_limit(limit)
    g = ctx.register_incidence(inc)
    p = ctx.plan(g, [1])
    st = p.stats()
    assert all(st[n] > 0 for n in slg.Plan.STAT_NAMES[1:8]), st
    p.destroy()
    for lg in ctx.line_graph(g, [1, 2, 9, 20]):
        ref = oracle.line_graph(inc, lg.s)
        for f, x in (("row_ptr", ref.row_ptr), ("row", ref.i), ("col", ref.j), ("w", ref.w)):
            np.testing.assert_array_equal(getattr(lg, f).cpu().numpy(), x, err_msg=f"{lg.s} {f}")
    g.release()
    ctx.close()
