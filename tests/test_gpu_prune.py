"""Pruning at its word edges: incidences and hyperedges on both sides of
multiples of 64 and of a wavefront's 512, first and last hyperedges kept or
dropped, nothing kept, empty lists at both ends, one threshold per row."""
from __future__ import annotations

import numpy as np
import pytest

import hypergen as hg
import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_2201_11326_amd as slg
    c = slg.Context(0)
    yield c
    c.close()


def sized(m, nnz, seed, n=97):
    """m hyperedges of 1..6 vertices with exactly nnz incidences; vertices 0
    and n - 1 are in none."""
    rng = np.random.default_rng(seed)
    size = np.full(m, nnz // m)
    size[rng.permutation(m)[:nnz - size.sum()]] += 1
    for _ in range(m):  # spread, keeping the sum
        a, b = rng.integers(0, m, 2)
        if size[a] > 1 and size[b] < 6:
            size[a] -= 1
            size[b] += 1
    rows = [np.sort(rng.choice(np.arange(1, n - 1), k, replace=False)) for k in size]
    return hg.from_csr(m, n, np.concatenate([[0], np.cumsum(size)]), np.concatenate(rows).astype(np.int32))


@pytest.mark.parametrize("m, nnz", [(1, 3), (21, 63), (21, 64), (22, 65), (63, 190), (64, 192), (65, 193), (170, 511),
                                    (170, 512), (171, 513), (640, 1920), (5000, 16_384), (5000, 16_385)])
@pytest.mark.parametrize("s", [2, 3, 7])
def test_pruned_lists(ctx, m, nnz, s):
    inc = sized(m, nnz, m + nnz)
    g = ctx.register_incidence(inc)
    for lg in ctx.line_graph(g, [s, s + 1]):
        ref = oracle.line_graph(inc, lg.s)
        np.testing.assert_array_equal(lg.row_ptr.cpu().numpy(), ref.row_ptr)
        np.testing.assert_array_equal(lg.col.cpu().numpy(), ref.j)
        np.testing.assert_array_equal(lg.w.cpu().numpy(), ref.w)
    g.release()


def test_pruned_by_a_threshold_per_row(ctx):
    incs = [sized(64 + i, 200 + 64 * i, i) for i in range(5)]
    graphs = [ctx.register_incidence(x) for x in incs]
    S = [1, 2, 3, 7, 2]
    b = ctx.batch(graphs, S)
    b.run()
    for i, (x, s) in enumerate(zip(incs, S)):
        lg, ref = b.result(i), oracle.line_graph(x, s)
        np.testing.assert_array_equal(lg.col.cpu().numpy(), ref.j)
        np.testing.assert_array_equal(lg.w.cpu().numpy(), ref.w)
    for g in graphs:
        g.release()
