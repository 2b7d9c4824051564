"""Infinities in the gradients: a row that gathers one is infinite, whatever surrounds it.  Places that a
kernel fills up (the end of a row, of a group) must not turn it into a NaN by multiplying it by zero."""
import numpy as np
import pytest
import torch

import graphgen
import oracle
import paper_2204_02662_amd as epp
from _util import ATOL, RTOL, dev, gpu_prepare, gpu_prepare_full, run_full, run_ifelse, run_partial

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


@pytest.mark.parametrize("layout", ["plain", "packed", "partitioned", "marked"])
@pytest.mark.parametrize("gs", [1, 3, 8, 24, 64])
@pytest.mark.parametrize("F", [2, 7, 16, 41, 64])
def test_groups_of_any_size(F, gs, layout, monkeypatch):
    """Group ends inside rows, right behind an infinite source; if-else baseline as well."""
    for k, v in {"EPP_TUNE_ROWS": "0", "EPP_TUNE_PACK": "2" if layout == "packed" else "0",
                 "EPP_TUNE_PART": "2" if layout == "partitioned" else "0", "EPP_TUNE_PART_KB": "16",
                 "EPP_TUNE_PART_MINLEN": "8", "EPP_TUNE_HOT_MB": "1" if layout == "marked" else "0"}.items():
        monkeypatch.setenv(k, v)
    g = graphgen.random_graph("rmat", 6_007, seed=51, raw_draws=60_000)  # (weights are positive)
    train = graphgen.training_set(g.n, 2_000, 52)
    sets_o, paths_o = oracle.prepare(g.n, g.rowptr, g.col, g.val, train, 1)
    paths, full = gpu_prepare(g, train, 1), gpu_prepare_full(g)
    src = np.flatnonzero(sets_o[0])
    X = _with_infinities(graphgen.normal_rows(g.n, F, sets_o[0], 53), src[::40])
    want = oracle.path_aggregate(g.n, paths_o[0], X)
    for p in (paths.path(0), full):
        p.set_group_size(F, gs)
    rows = sets_o[1].astype(bool)
    _assert_same(run_partial(paths.path(0), X)[rows], want[rows], f"F={F} gs={gs}")
    _assert_same(run_ifelse(full, paths, 0, X)[rows], want[rows], f"if-else F={F} gs={gs}")
    _assert_same(run_full(full, X), oracle.full_aggregate(g.n, g.rowptr, g.col, g.val, X), f"all-active F={F} gs={gs}")
