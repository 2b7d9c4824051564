"""Preparation of graphs whose bitmap does not fit LDS: windows of it, one pass over groups of four or eight ids, and lookups
(few entries, or more than 10.2 M ids); sets that are sparse, dense, and neither."""
import functools

import numpy as np
import pytest
import torch

import oracle
import paper_2204_02662_amd as epp
from _util import assert_paths_bit_exact, dev

pytestmark = pytest.mark.gpu

WINDOW = 39_936 * 32  # ids


@functools.lru_cache(maxsize=1)
def _graph(n, entries, seed):
    """Entries of the first, the last and random vertices; no entry elsewhere."""
    rng = np.random.default_rng(seed)
    ends = np.concatenate([np.arange(70), np.arange(n - 70, n), np.arange(WINDOW - 5, WINDOW + 5)])
    row = np.concatenate([rng.integers(0, n, entries - 10_000), rng.choice(ends, 10_000)])
    col = np.concatenate([rng.integers(0, n, entries - 20_000), rng.choice(ends, 20_000)])
    pairs = np.unique(row.astype(np.int64) * n + col)
    rowptr = np.searchsorted(pairs, np.arange(n + 1, dtype=np.int64) * n).astype(np.int32)
    col = (pairs % n).astype(np.int32)
    return rowptr, col, rng.standard_normal(col.size).astype(np.float32)


@pytest.mark.parametrize("percent", [2, 50, 97])
@pytest.mark.parametrize("n,entries", [(2 * WINDOW + 1, 300_000), (3 * WINDOW, 300_000), (3 * WINDOW + 1, 300_000),
                                       (3 * WINDOW + 1, 6_100_000), (4 * WINDOW + 1, 6_100_000), (8 * WINDOW, 6_100_000),
                                       (8 * WINDOW + 3, 6_100_000)])
def test_paths_and_columns_out_of_range(n, entries, percent):
    rowptr, col, val = _graph(n, entries, 17)
    rng = np.random.default_rng(18)
    train = np.flatnonzero(rng.random(n) < percent / 100).astype(np.int32)
    train = np.union1d(train, [0, n - 1, WINDOW]).astype(np.int32)
    d = dev()
    up = [torch.from_numpy(x).to(d) for x in (rowptr, col, val, train)]
    sets_o, paths_o = oracle.prepare(n, rowptr, col, val, train, 2)
    assert_paths_bit_exact(epp.epp_prepare(n, *up, 2), sets_o, paths_o, 2)
    for bad in (n, -1, 2**31 - 1):
        wrong = up[1].clone()
        wrong[1234] = bad
        with pytest.raises(Exception, match="outside"):
            epp.epp_prepare(n, up[0], wrong, up[2], up[3], 2)
