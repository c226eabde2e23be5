"""The two-pass transpose behind the symmetric CSR at its edges: digit widths
(vertex counts around powers of two, the most that pack and one more), tiles of
8192 items and chunks, rows that fill wavefronts and single-entry rows, columns
that share digits, and inputs whose rows start or end elsewhere than their
pointers say."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from test_gpu_symmetric import _Edges, _check

pytestmark = pytest.mark.gpu

TILE = 8192


@pytest.fixture(scope="module")
def ctx():
    import paper_2201_11326_amd as slg
    c = slg.Context(0)
    yield c
    c.close()


def exactly(m, n, seed, dense_rows=0):
    """n distinct edges of m vertices in CSR order; the first `dense_rows`
    rows hold every later vertex."""
    rng = np.random.default_rng(seed)
    keys = [r * m + np.arange(r + 1, m, dtype=np.int64) for r in range(dense_rows)]
    key = np.unique(np.concatenate(keys)) if keys else np.empty(0, np.int64)
    while key.size < n:
        a, b = rng.integers(0, m, n), rng.integers(0, m, n)
        k = np.minimum(a, b) * m + np.maximum(a, b)
        key = np.unique(np.concatenate([key, k[a != b]]))
    if key.size > n:
        key = np.sort(rng.permutation(key)[:n]) if not dense_rows else key[:n]
    row, col = (key // m).astype(np.int32), (key % m).astype(np.int32)
    row_ptr = np.concatenate([[0], np.cumsum(np.bincount(row, minlength=m))]).astype(np.int64)
    return row_ptr, row, col, rng.integers(1, 1 << 30, n).astype(np.int32)


@pytest.mark.parametrize("m", [2, 3, 4, 5, 1 << 9, (1 << 9) + 1, (1 << 18) - 1, 1 << 18, (1 << 18) + 1, 1 << 20,
                               (1 << 20) + 1])
@pytest.mark.parametrize("n", [1, 63, 64, 65, TILE - 1, TILE, TILE + 1, 3 * TILE + 17])
def test_vertex_and_item_counts(ctx, m, n):
    n = min(n, m * (m - 1) // 2)
    _check(ctx, m, *exactly(m, n, m + n))


@pytest.mark.parametrize("weights", [True, False])
def test_long_rows_and_many_tiles_per_chunk(ctx, weights):
    """2.5e7 items: three tiles per chunk; whole rows beside sparse ones."""
    _check(ctx, 60_000, *exactly(60_000, 3 * 1024 * TILE + 12_345, 5, dense_rows=100), weights=weights)


def test_rows_that_start_or_end_elsewhere(ctx):
    import paper_2201_11326_amd as slg
    m, n = 5000, 2 * TILE + 100
    row_ptr, row, col, w = exactly(m, n, 11)
    cases = []
    for e in (1, 64, TILE, n - 1):  # the run of a row one entry short or long of its pointers
        e = int(np.flatnonzero(np.diff(row[:e + 1], prepend=-1))[-1])
        for d in (-1, 1):
            p = row_ptr.copy()
            p[row[e]] += d
            cases.append((p, row, col))
    r = row.copy()
    r[-1] = min(int(r[-1]) + 1, int(col[-1]) - 1)
    if r[-1] != row[-1]:
        cases.append((row_ptr, r, col))
    for bad in (-1, m, 2**31 - 1, -2**31):
        for at in (0, TILE, n - 1):
            c = col.copy()
            c[at] = bad
            cases.append((row_ptr, row, c))
            r = row.copy()
            r[at] = bad
            cases.append((row_ptr, r, col))
    for p, r, c in cases:
        with pytest.raises(slg.SlgError) as ei:
            ctx.symmetrize(_Edges(p, r, c, w))
        assert ei.value.status == slg.SLG_ERR_INVALID_ARG
    _check(ctx, m, row_ptr, row, col, w)
