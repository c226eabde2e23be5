"""The light tier on both sides of the sizes where its launches change (16384
rows of the sorting classes counted together or by class; 2^24 2-paths for the
store laid out by every row's), with and without its store, against the
oracle."""
from __future__ import annotations

import numpy as np
import pytest

import hypergen as hg
import oracle

pytestmark = pytest.mark.gpu


def band(m, width):
    """Row i holds vertices i .. i + width - 1: it shares width - d with row
    i + d, and every row but the last few has width * (width - 1) / 2 2-paths."""
    ptr = np.arange(m + 1, dtype=np.int64) * width
    idx = (np.arange(m)[:, None] + np.arange(width)).astype(np.int32).ravel()
    return hg.from_csr(m, m + width - 1, ptr, idx)


# width 5: ten 2-paths a row, more than eight in all rows but the last three;
# width 12: 66, the next class; width 23 on 2^16 rows: 253 a row, 2^24 - 1 of
# them at most 66 312 rows
@pytest.mark.parametrize("m, width", [(16_386, 5), (16_387, 5), (16_388, 5), (3, 5), (16_000, 12), (40_000, 3),
                                      (66_000, 23), (66_600, 23)])
@pytest.mark.parametrize("store", [True, False])
def test_light_rows(m, width, store):
    import paper_2201_11326_amd as slg
    ctx = slg.Context(0)
    if not store:
        ctx.set_count_store(0)
    inc = band(m, width)
    g = ctx.register_incidence(inc)
    S = [1, 2, 4]
    for lg in ctx.line_graph(g, S):
        ref = oracle.line_graph(inc, lg.s)
        np.testing.assert_array_equal(lg.row_ptr.cpu().numpy(), ref.row_ptr)
        np.testing.assert_array_equal(lg.col.cpu().numpy(), ref.j)
        np.testing.assert_array_equal(lg.w.cpu().numpy(), ref.w)
        np.testing.assert_array_equal(lg.row.cpu().numpy(), ref.i)
    g.release()
    ctx.close()
