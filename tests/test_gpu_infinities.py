"""Infinities in the gradients: a row that gathers one is infinite, whatever surrounds it.  Places that a
kernel fills up (the end of a row, of a group) must not turn it into a NaN by multiplying it by zero."""
import numpy as np
import pytest
import torch

import graphgen
import oracle
import paper_2204_02662_amd as epp
from _util import ATOL, RTOL, dev, gpu_prepare, run_partial

pytestmark = pytest.mark.gpu


def _assert_same(got, want, what):
    inf = ~np.isfinite(want)
    assert inf.any()
    assert np.array_equal(got[inf], want[inf].astype(np.float32)), what
    assert np.all(np.abs(got[~inf] - want[~inf]) <= ATOL + RTOL * np.abs(want[~inf])), what


def _with_infinities(X, ids):
    """+Inf in one column or another of the given rows."""
    X[ids, np.arange(ids.size) % X.shape[1]] = np.inf
    return X


@pytest.mark.parametrize("F", [1, 2, 3, 4, 7, 16, 41, 64, 130])
def test_row_kernel(F, monkeypatch):
    """The last source of every row is infinite; rows of every length modulo the step, up to cut ones."""
    monkeypatch.setenv("EPP_TUNE_ROWS", "2")
    lanes = 1
    while 4 * lanes < F and lanes < 64:
        lanes *= 2
    lengths = np.concatenate([np.arange(1, 140), 8192 // lanes + np.arange(-3, 6), [2 * 8192 // lanes + 1]])
    m = lengths.size
    n = int(lengths.max()) + m  # the last m vertices are the rows' last sources, one each
    rng = np.random.default_rng(5)
    col = np.concatenate([np.r_[np.sort(rng.choice(n - m, size=k - 1, replace=False)), n - m + r]
                          for r, k in enumerate(lengths)]).astype(np.int32)
    rowptr = np.zeros(n + 1, np.int32)
    rowptr[1:m + 1] = np.cumsum(lengths)
    rowptr[m + 1:] = rowptr[m]
    # (a row's |w x| add up to 1/4 at most on average and 40 additions follow each other at most: the finite results
    # are within 40 * 2^-24 / 4 = 6e-7 of the exact ones)
    val = ((rng.random(col.size) + 0.1) / (2 * np.repeat(lengths, lengths))).astype(np.float32)
    train = np.arange(n, dtype=np.int32)
    sets_o, paths_o = oracle.prepare(n, rowptr, col, val, train, 1)
    paths = epp.epp_prepare(n, *(torch.from_numpy(a).to(dev()) for a in (rowptr, col, val, train)), 1)
    X = _with_infinities(graphgen.normal_rows(n, F, sets_o[0], 6), np.arange(n - m, n))
    want = oracle.path_aggregate(n, paths_o[0], X)
    assert np.isinf(want[:m]).any(1).all()
    p = paths.path(0)
    p.prepare_width(F)
    _assert_same(run_partial(p, X)[:m], want[:m], f"F={F}")


@pytest.mark.parametrize("F", [3, 16, 64])
def test_inner_path_does_not_meet_the_weights_of_the_outer_one(F, monkeypatch):
    """Entries of the outer path only may have any weight: the inner path skips them."""
    monkeypatch.setenv("EPP_TUNE_ROWS", "2")
    monkeypatch.setenv("EPP_TUNE_SHARE_PCT", "1")
    monkeypatch.setenv("EPP_TUNE_SMALL_PREPARE", "0")
    g = graphgen.random_graph("rmat", 20_011, seed=31, raw_draws=250_000)
    train = graphgen.training_set(g.n, 600, 32)
    sets_o, paths_o = oracle.prepare(g.n, g.rowptr, g.col, g.val, train, 2)
    g.val[sets_o[0][g.col] == 0] = np.inf
    paths = gpu_prepare(g, train, 2)
    assert paths.path(1).info().shares_entries == 1
    X = graphgen.normal_rows(g.n, F, sets_o[0], 33)
    want = oracle.path_aggregate(g.n, paths_o[1], X)
    got = run_partial(paths.path(1), X)
    assert np.all(np.abs(got - want) <= ATOL + RTOL * np.abs(want))
