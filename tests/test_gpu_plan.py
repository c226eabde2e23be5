"""The planning kernels through the C ABI at their edges: the per-row 2-path
work (work prefix) of whole graphs against the oracle, row counts on both
sides of the wavefront group's sizes, member counts around the small-row and
piece bounds, and malformed vertex lists found wherever they are."""
from __future__ import annotations

import numpy as np
import pytest

import hypergen as hg
import oracle

pytestmark = pytest.mark.gpu

SIZES = [0, 1, 2, 15, 16, 17, 63, 64, 65, 66, 255, 256, 257, 511, 512, 513, 700]


def sized(m, n, seed):
    """m rows, most of 0..9 members, every 50th of a size around the bounds."""
    rng = np.random.default_rng(seed)
    size = rng.integers(0, 10, m)
    size[::50] = rng.choice(SIZES, size[::50].size)
    row = np.repeat(np.arange(m), size)
    key = np.unique(row * n + (rng.random(row.size) ** 2 * n).astype(np.int64))
    he_ptr = np.concatenate([[0], np.cumsum(np.bincount(key // n, minlength=m))])
    return hg.from_csr(m, n, he_ptr, (key % n).astype(np.int32))


def row_work(inc, s):
    """2-paths e_i -> v -> e_j, j > i, per row i: what follows i in each of
    its members' lists of hyperedges with at least s members."""
    v = np.repeat(np.arange(inc.n), np.diff(inc.v_ptr))
    e = inc.v_idx.astype(np.int64)
    keep = inc.sizes()[e] >= s
    v, e = v[keep], e[keep]
    end = np.concatenate([np.nonzero(np.diff(v))[0], [v.size - 1]]) if v.size else v
    last = np.zeros(inc.n, np.int64)
    last[v[end]] = end
    return np.bincount(e, weights=last[v] - np.arange(v.size), minlength=inc.m).astype(np.int64)


@pytest.fixture(scope="module")
def ctx():
    import paper_2201_11326_amd as slg
    c = slg.Context(0)
    yield c
    c.close()


# 1, 15..17, 63..65: rows of one or two wavefront groups; 2^17: where the
# group grows from 16 to 64 rows
@pytest.mark.parametrize("m", [1, 15, 16, 17, 63, 64, 65, 1000, (1 << 17) - 1, 1 << 17, (1 << 17) + 65])
@pytest.mark.parametrize("s", [1, 3])
def test_work_prefix_equals_oracle(ctx, m, s):
    inc = sized(m, max(m // 3, 900), seed=m + s)
    g = ctx.register_incidence(inc)
    pre = ctx.work_prefix(g, s)
    assert pre[0] == 0
    np.testing.assert_array_equal(np.diff(pre), row_work(inc, s))
    if m <= 1000:
        np.testing.assert_array_equal(np.diff(pre), oracle.row_two_paths(inc, s, np.arange(m)))
    g.release()


@pytest.mark.parametrize("m", [2000, (1 << 17) + 7])
@pytest.mark.parametrize("member", ["first", "last", "large"])
def test_malformed_vertex_list_is_found(ctx, m, member):
    """An incidence that the vertex CSR lacks: planning reports the graph."""
    import torch
    import paper_2201_11326_amd as slg
    inc = sized(m, m, seed=5)
    sz = inc.sizes()
    big = int(np.nonzero(sz > 300)[0][-1])
    p = {"first": 0, "last": inc.nnz - 1, "large": int(inc.he_ptr[big]) + 299}[member]
    i = int(np.searchsorted(inc.he_ptr, p, side="right")) - 1
    v = int(inc.he_idx[p])
    v_idx = inc.v_idx.copy()
    at = int(inc.v_ptr[v]) + int(np.searchsorted(v_idx[inc.v_ptr[v]:inc.v_ptr[v + 1]], i))
    assert v_idx[at] == i
    v_idx[at] = max(i - 1, 0) if i else 1
    t = lambda a, dt: torch.as_tensor(a, dtype=dt).cuda()
    g = ctx.register(inc.m, inc.n, t(inc.he_ptr, torch.int64), t(inc.he_idx, torch.int32), t(inc.v_ptr, torch.int64),
                     t(v_idx, torch.int32))
    with pytest.raises(slg.SlgError) as ei:
        ctx.line_graph(g, [1])
    assert ei.value.status == slg.SLG_ERR_INVALID_GRAPH
    g.release()
