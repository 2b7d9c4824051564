"""Graphs whose rows are as uneven as they can be: millions of vertices without entries between a few with some, one row
that holds a third of all entries.  Paths bit for bit, and aggregation over the tables made for them."""
import numpy as np
import pytest
import torch

import graphgen
import oracle
import paper_2204_02662_amd as epp
from _util import assert_close, assert_paths_bit_exact, dev, run_partial

pytestmark = pytest.mark.gpu


def _csr(n, u, v, seed):
    keys = np.unique(u.astype(np.int64) * n + v)
    rowptr = np.zeros(n + 1, np.int32)
    rowptr[1:] = np.cumsum(np.bincount(keys // n, minlength=n))
    val = np.random.default_rng(seed).standard_normal(keys.size).astype(np.float32) / 64
    return n, rowptr, (keys % n).astype(np.int32), val


def _gaps(rng):
    """Directed; clusters of rows at both ends and in the middle, everything else empty."""
    n = 700_001
    at = np.concatenate([np.arange(3_000), 350_000 + 97 * np.arange(1_000), n - 1 - np.arange(2_000)])
    return _csr(n, rng.choice(at, 90_000), rng.choice(at, 90_000), 1)


def _star(rng):
    """One row of 200,000 entries (more than sixty tiles), in the middle of the ids, and one vertex in all rows."""
    n = 200_001
    ids, hub = np.arange(n), np.full(n, n // 2)
    return _csr(n, np.concatenate([ids, hub, ids]), np.concatenate([hub, ids, ids]), 2)


def _long_rows(rng):
    """Long rows that most levels filter to little, beside empty and short ones."""
    n = 90_000
    u = np.concatenate([np.repeat(rng.integers(0, n, 40), 5_000), rng.integers(0, n, 60_000)])
    return _csr(n, u, rng.integers(0, n, u.size), 3)


@pytest.mark.parametrize("share", ["0", "95"])
@pytest.mark.parametrize("shape", [_gaps, _star, _long_rows])
def test_paths(shape, share, monkeypatch):
    monkeypatch.setenv("EPP_TUNE_SHARE_PCT", share)
    monkeypatch.setenv("EPP_TUNE_SMALL_PREPARE", "0")
    n, rowptr, col, val = shape(np.random.default_rng(7))
    g = tuple(torch.from_numpy(a).to(dev()) for a in (rowptr, col, val))
    some = np.random.default_rng(8).choice(np.unique(col), 50, replace=False).astype(np.int32)
    for train in (some, some[:1], np.arange(n, dtype=np.int32)):
        sets_o, paths_o = oracle.prepare(n, rowptr, col, val, train, 3)
        paths = epp.epp_prepare(n, *g, torch.from_numpy(train).to(dev()), 3)
        assert_paths_bit_exact(paths, sets_o, paths_o, 3)


@pytest.mark.parametrize("rows", ["0", "2"])
@pytest.mark.parametrize("F", [1, 4, 16, 64])
def test_aggregation_over_a_star(F, rows, monkeypatch):
    monkeypatch.setenv("EPP_TUNE_ROWS", rows)
    n, rowptr, col, val = _star(None)
    train = np.arange(n, dtype=np.int32)
    sets_o, paths_o = oracle.prepare(n, rowptr, col, val, train, 1)
    paths = epp.epp_prepare(n, *(torch.from_numpy(a).to(dev()) for a in (rowptr, col, val, train)), 1)
    X = graphgen.normal_rows(n, F, sets_o[0], 9)
    p = paths.path(0)
    if rows == "0":
        p.set_group_size(F, 64)
    else:
        p.prepare_width(F)
    got, want = run_partial(p, X), oracle.path_aggregate(n, paths_o[0], X)
    others = np.arange(n) != n // 2
    assert_close(got[others], want[others], f"F={F}")
    # the hub adds 200,000 terms of standard deviation 1/64: at most 2,000 of them follow each other in 32 bits
    assert np.all(np.abs(got[n // 2] - want[n // 2]) <= 2000 * 2.0 ** -24 * np.sqrt(n) / 64 * 4)
