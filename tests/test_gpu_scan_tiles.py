"""Prefix sums by one workgroup at the edge of its first tile (512 threads of
eight entries), where a second one starts: rows, slots and kept words."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from test_gpu_scan import chain

pytestmark = pytest.mark.gpu

TILE = 512 * 8


@pytest.mark.parametrize("m", [TILE - 1, TILE, TILE + 1, TILE + 2, 2 * TILE - 1])
@pytest.mark.parametrize("k", [1, 16])
def test_rows_and_slots_at_the_tile_edge(m, k):
    import paper_2201_11326_amd as slg
    ctx = slg.Context(0)
    inc = chain(m, max(1, m // 9))
    s_list = list(range(1, k + 1))
    g = ctx.register_incidence(inc)
    for s, lg in zip(s_list, ctx.line_graph(g, s_list)):
        ref = oracle.line_graph(inc, s)
        for f, x in (("row_ptr", ref.row_ptr), ("col", ref.j), ("w", ref.w)):
            np.testing.assert_array_equal(getattr(lg, f).cpu().numpy(), x, err_msg=f"{s} {f}")
    g.release()
    ctx.close()


@pytest.mark.parametrize("words", [TILE - 1, TILE, TILE + 1])
@pytest.mark.parametrize("spare", [-1, 0, 1])
def test_kept_words_at_the_tile_edge(words, spare):
    """64 * words incidences, one more and one less: two kept rows at either
    end of a hypergraph of rows that s = 3 prunes."""
    import hypergen as hg
    import paper_2201_11326_amd as slg
    nnz = 64 * words + spare
    small = nnz - 12  # incidences in rows of one vertex
    n = small + 4
    ptr = np.concatenate([[0, 3, 6], 6 + np.arange(1, small + 1), [nnz - 3, nnz]])
    idx = np.concatenate([[0, 1, n - 1, 0, 1, 2], np.arange(2, small + 2), [0, 1, n - 1, 2, n - 2, n - 1]])
    inc = hg.from_csr(ptr.size - 1, n, ptr.astype(np.int64), idx.astype(np.int32))
    ctx = slg.Context(0)
    g = ctx.register_incidence(inc)
    lg = ctx.line_graph(g, [3])[0]
    kept = [0, 1, inc.m - 2, inc.m - 1]
    ref = oracle.line_graph_rows(inc, 3, kept)
    assert lg.num_edges == sum(ref.row(t)[0].size for t in range(len(kept))) == 1
    assert (int(lg.row[0]), int(lg.col[0]), int(lg.w[0])) == (0, inc.m - 2, 3)
    g.release()
    ctx.close()
