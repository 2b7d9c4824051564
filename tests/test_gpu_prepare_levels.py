"""Paths of up to seven layers whose sets grow slowly, so that most levels have entries of their own: the entries of a level
are written by the pass that writes those of a later one, whichever levels share theirs."""
import numpy as np
import pytest

import graphgen
import oracle
from _util import assert_close, assert_paths_bit_exact, gpu_prepare, run_partial

pytestmark = pytest.mark.gpu


class _Ring:
    """Every vertex next to four others on a ring of shuffled ids, with or without itself; one row is longer than a tile."""

    def __init__(self, n, loops, seed):
        rng = np.random.default_rng(seed)
        order = rng.permutation(n)
        steps = (-2, -1, 0, 1, 2) if loops else (-3, -1, 1, 2)
        row = np.concatenate([order] * len(steps) + [np.full(5_000, order[7])])
        col = np.concatenate([order[(np.arange(n) + s) % n] for s in steps] + [rng.choice(n, 5_000, replace=False)])
        pairs = np.unique(row.astype(np.int64) * n + col)
        self.n, self.col = n, (pairs % n).astype(np.int32)
        self.rowptr = np.searchsorted(pairs, np.arange(n + 1, dtype=np.int64) * n).astype(np.int32)
        # (values of a normalised graph: a row's terms then add up to |w x| <= sqrt(5,000) at most, in 5,000 / 32 + 32 additions
        # that round by 2^-24 each, 1e-6 in the root mean square; values of one would take the long row's error to 70 times that)
        lens = np.diff(self.rowptr)
        self.val = (rng.standard_normal(self.col.size) / np.sqrt(np.repeat(lens, lens))).astype(np.float32)


@pytest.mark.parametrize("share", ["0", "60", "75", "95"])
@pytest.mark.parametrize("loops", [True, False])
def test_levels_of_their_own(loops, share, monkeypatch):
    for k, v in {"SMALL_PREPARE": "0", "SHARE_PCT": share, "ROWS": "0"}.items():
        monkeypatch.setenv("EPP_TUNE_" + k, v)
    g = _Ring(20_011, loops, 91)
    train = np.sort(np.random.default_rng(92).choice(g.n, 300, replace=False)).astype(np.int32)
    for L in (1, 2, 3, 4, 7):
        sets_o, paths_o = oracle.prepare(g.n, g.rowptr, g.col, g.val, train, L)
        paths = gpu_prepare(g, train, L)
        assert_paths_bit_exact(paths, sets_o, paths_o, L)
        for l in range(L):  # (the group kernel goes by the row-end marks)
            X = graphgen.normal_rows(g.n, 16, sets_o[L - 1 - l], 93 + l)
            assert_close(run_partial(paths.path(l), X), oracle.path_aggregate(g.n, paths_o[l], X), f"L={L} l={l}")
