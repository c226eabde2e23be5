"""Tiny rows on both sides of the number from which they are counted apart
from the sorting classes (3 * 2^20), with and without the light store, against the
overlaps of the bands that the input is made of and oracle rows."""
from __future__ import annotations

import numpy as np
import pytest

import hypergen as hg
import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tiny", [3 << 20, (3 << 20) + 1])
@pytest.mark.parametrize("store", [True, False])
def test_tiny_rows_beside_sorting_rows(tiny, store):
    import paper_2201_11326_amd as slg
    # bands of rows i .. i + width - 1: a row of the first has three 2-paths (the
    # last two have two and none), one of the second 66 (the last five 45 to none)
    ptr, idx, at, e = [np.zeros(1, np.int64)], [], 0, 0
    for width, rows in ((3, tiny + 1), (12, 50)):
        idx.append((at + np.arange(rows)[:, None] + np.arange(width)).astype(np.int32).ravel())
        ptr.append(e + width * np.arange(1, rows + 1, dtype=np.int64))
        e += width * rows
        at += rows + width
    ptr = np.concatenate(ptr)
    inc = hg.from_csr(ptr.size - 1, at, ptr, np.concatenate(idx))
    ctx = slg.Context(0)
    if not store:
        ctx.set_count_store(0)
    g = ctx.register_incidence(inc)
    p = ctx.plan(g, [1])
    st = p.stats()
    p.destroy()
    assert st["tiny8"] == tiny and st["light64"] > 0 and st["light128"] > 0, st
    first = tiny + 1  # rows of the first band
    for lg in ctx.line_graph(g, [1, 2, 5]):
        # row i of a band shares width - d vertices with row i + d
        want = []
        for width, lo, hi in ((3, 0, first), (12, first, inc.m)):
            d = np.arange(1, width - lg.s + 1)
            i = np.repeat(np.arange(lo, hi), d.size)
            j = i + np.tile(d, hi - lo)
            want.append((i[j < hi], j[j < hi], (width - (j - i))[j < hi]))
        row, col, w = (np.concatenate(x) for x in zip(*want))
        for f, x in (("row", row), ("col", col), ("w", w),
                     ("row_ptr", np.concatenate([[0], np.cumsum(np.bincount(row, minlength=inc.m))]))):
            np.testing.assert_array_equal(getattr(lg, f).cpu().numpy(), x, err_msg=f"{lg.s} {f}")
        ref = oracle.line_graph_rows(inc, lg.s, [0, first - 3, first - 1, first, inc.m - 2])
        for t, r in enumerate(ref.rows):
            rj, rw = ref.row(t)
            assert np.array_equal(col[row == r], rj) and np.array_equal(w[row == r], rw), int(r)
    g.release()
    ctx.close()
