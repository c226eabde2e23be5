"""Edge lists that slg_symmetrize refuses, past the ones of
test_gpu_symmetric.py."""
from __future__ import annotations

import numpy as np
import pytest

import hypergen as hg
from test_gpu_symmetric import _Edges, _check

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_2201_11326_amd as slg
    c = slg.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("edges", [1, 300, 1 << 20])
def test_edges_without_vertices(ctx, edges):
    import paper_2201_11326_amd as slg
    e = np.arange(edges, dtype=np.int32)
    for weights in (True, False):
        with pytest.raises(slg.SlgError) as ei:
            ctx.symmetrize(_Edges(np.zeros(1, np.int64), e, e + 1, e), weights=weights)
        assert ei.value.status == slg.SLG_ERR_INVALID_ARG and "upper triangle" in str(ei.value)
    _check(ctx, 1000, *hg.random_upper_edges(9, 1000, 20000, 1.0))


@pytest.mark.parametrize("weights", [True, False])
def test_rows_that_overlap_are_not_copied(ctx, weights):
    """Long rows (256 entries and more on average) whose pointers alternate
    between 0 and n: each would be all of the list. The call fails, and what
    it has written by then is at most the lower parts, one place per edge."""
    import ctypes
    import torch
    import paper_2201_11326_amd as slg
    m = 600
    row, col = (x.astype(np.int32) for x in np.triu_indices(m, 1))
    n = row.size
    assert n // m >= 256
    ptr = np.zeros(m + 1, np.int64)
    ptr[1::2] = n
    ptr[m] = n
    good = np.concatenate([[0], np.cumsum(np.bincount(row, minlength=m))])
    e = _Edges(ptr, row, col, np.ones(n, np.int32))
    sym_ptr = torch.empty(m + 1, dtype=torch.int64, device="cuda")
    out = [torch.full((2 * n,), -7, dtype=torch.int32, device="cuda") for _ in range(2)]
    status = slg.lib().slg_symmetrize(ctx.handle, m, e.row_ptr.data_ptr(), e.row.data_ptr(), e.col.data_ptr(),
                                      e.w.data_ptr() if weights else None, n, sym_ptr.data_ptr(), out[0].data_ptr(),
                                      out[1].data_ptr() if weights else None, ctypes.c_void_p(0))
    torch.cuda.synchronize()
    assert status == slg.SLG_ERR_INVALID_ARG
    for o in out[:2 if weights else 1]:
        assert int((o != -7).sum()) <= n
    _check(ctx, m, good, row, col, np.ones(n, np.int32), weights=weights)
