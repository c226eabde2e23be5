"""Prefix sums at the sizes where their launches change: one workgroup per
array up to 32768 entries (in tiles of 8192), three launches for all arrays
beyond (tiles of 4096), one to sixteen arrays of one call."""
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


def chain(m, extra):
    """Row i holds vertices i and i + 1, and row i with i % 3 == 0 one of
    `extra` more: every row but the last has one slot, so slots count to m - 1."""
    rows = np.repeat(np.arange(m), 2 + (np.arange(m) % 3 == 0))
    ptr = np.concatenate([[0], np.cumsum(np.bincount(rows, minlength=m))])
    idx = np.empty(rows.size, np.int32)
    idx[ptr[:-1]] = np.arange(m)
    idx[ptr[:-1] + 1] = np.arange(m) + 1
    third = np.arange(0, m, 3)
    idx[ptr[third] + 2] = m + 1 + third // 3 % extra
    return hg.from_csr(m, m + 1 + extra, ptr, idx)


@pytest.mark.parametrize("m", [1, 2, 8192, 8193, 8194, 32767, 32768, 32769, 32770, 36865, 65537])
@pytest.mark.parametrize("k", [1, 3, 16])
def test_prefix_sums_at_launch_edges(ctx, m, k):
    inc = chain(m, max(1, m // 9))
    s_list = list(range(1, k + 1))
    g = ctx.register_incidence(inc)
    outs = ctx.line_graph(g, s_list)
    for s, lg in zip(s_list, outs):
        ref = oracle.line_graph(inc, s)
        np.testing.assert_array_equal(lg.row_ptr.cpu().numpy(), ref.row_ptr)
        np.testing.assert_array_equal(lg.col.cpu().numpy(), ref.j)
        np.testing.assert_array_equal(lg.w.cpu().numpy(), ref.w)
    pre = ctx.work_prefix(g, 1)
    assert pre[0] == 0 and pre.size == m + 1 and np.all(np.diff(pre) >= 0)
    if k == 1:
        # every shared vertex is one 2-path: the sum of weights at s = 1
        assert pre[-1] == int(outs[0].w.sum())
    g.release()
