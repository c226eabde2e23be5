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
