"""A server whose budget is exactly what a query needs without the stores that
small plans keep by themselves: the query still succeeds, at once or in a
second attempt, within the budget."""
from __future__ import annotations

import pytest

import hypergen as hg
from gpu_util import assert_matches_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("spare", [0, 1 << 30])
def test_budget_without_room_for_small_stores(spare):
    import paper_2201_11326_amd as slg
    inc = hg.random_small(9, 3000, 1500, 40)
    S = [1, 2, 4]

    def ask(stores, budget):
        ctx = slg.Context(0)
        if not stores:
            ctx.set_count_store(32 << 30, 1 << 24)
        g = ctx.register_incidence(inc)
        srv = ctx.server(workers=1, mem_budget_bytes=budget)
        r = srv.wait(srv.submit(g, S), timeout_ms=60_000)
        assert r is not None and r.ok, r and r.message
        attempts, got = r.attempts, [lg.cpu() for lg in r.outs]
        del r
        st = srv.stats()
        assert st["bytes_used"] == 0 and st["failed"] == 0
        srv.close()
        g.release()
        ctx.close()
        for lg in got:
            assert_matches_oracle(inc, lg, lg.s)
        return st["bytes_peak"], attempts

    need, attempts = ask(False, 0)
    assert attempts == 1
    more, _ = ask(True, 0)
    assert more > need
    peak, attempts = ask(True, need + spare)
    assert peak <= need + spare and attempts == (1 if spare else 2)
