"""The kernel that processes rows whole (small paths, narrow rows): rows at the lengths where it changes
its way (one step of a slot, left to the workgroup, cut into chunks), at every shape of a source row."""
import numpy as np
import pytest
import torch

import graphgen
import oracle
import paper_2204_02662_amd as epp
from _util import assert_close, dev, gpu_prepare, run_partial

pytestmark = pytest.mark.gpu

# one float per lane group up to 256 and beyond (two column windows)
WIDTHS = [1, 2, 3, 4, 5, 7, 16, 17, 41, 64, 127, 128, 256, 259]


def _graph_with_rows(lengths, n, seed):
    """n vertices, row i has lengths[i] distinct sources (the rest of the rows: one)."""
    rng = np.random.default_rng(seed)
    lens = np.ones(n, np.int64)
    at = rng.permutation(n)[:len(lengths)]
    lens[at] = lengths
    rowptr = np.zeros(n + 1, np.int32)
    rowptr[1:] = np.cumsum(lens)
    col = np.concatenate([np.sort(rng.choice(n, size=k, replace=False)) for k in lens]).astype(np.int32)
    val = (rng.standard_normal(col.size) / np.sqrt(np.repeat(lens, lens))).astype(np.float32)
    return n, rowptr, col, val


@pytest.mark.parametrize("F", WIDTHS)
def test_rows_of_every_length_class(F, monkeypatch):
    monkeypatch.setenv("EPP_TUNE_ROWS", "2")
    lanes = 1
    while 4 * lanes < F and lanes < 64:
        lanes *= 2
    chunk = 8192 // lanes
    lengths = [2, 3, 4, 5, 8, 9, 31, 32, 33, 63, 64, 65, 127, 128, 129, chunk - 1, chunk, chunk + 1, 2 * chunk,
               2 * chunk + 1, 3 * chunk - 5]
    n, rowptr, col, val = _graph_with_rows(lengths, 3 * chunk + 500, 11)
    train = np.arange(n, dtype=np.int32)
    sets_o, paths_o = oracle.prepare(n, rowptr, col, val, train, 1)
    d = dev()
    paths = epp.epp_prepare(n, *(torch.from_numpy(a).to(d) for a in (rowptr, col, val, train)), 1)
    X = graphgen.normal_rows(n, F, sets_o[0], 12)
    want = oracle.path_aggregate(n, paths_o[0], X)
    p = paths.path(0)
    p.prepare_width(F)
    got = run_partial(p, X)
    assert_close(got, want, f"F={F}")
    assert np.array_equal(got, run_partial(p, X))  # equal inputs, equal bits
    assert p.info().n_split_rows == 0


@pytest.mark.parametrize("F", [3, 16, 47, 300])
def test_rows_of_an_inner_path_on_the_outer_paths_entries(F, monkeypatch):
    """Entries that are not the inner path's are skipped and never read, in short, long and cut rows."""
    monkeypatch.setenv("EPP_TUNE_ROWS", "2")
    monkeypatch.setenv("EPP_TUNE_SHARE_PCT", "1")
    monkeypatch.setenv("EPP_TUNE_SMALL_PREPARE", "0")
    g = graphgen.random_graph("rmat", 30_011, seed=77, raw_draws=400_000)
    train = graphgen.training_set(g.n, 900, 78)
    sets_o, paths_o = oracle.prepare(g.n, g.rowptr, g.col, g.val, train, 2)
    paths = gpu_prepare(g, train, 2)
    assert paths.path(1).info().shares_entries == 1
    for l in (1, 0):
        X = graphgen.normal_rows(g.n, F, sets_o[1 - l], 79 + l)
        want = oracle.path_aggregate(g.n, paths_o[l], X)
        X[sets_o[1 - l] == 0] = np.nan
        p = paths.path(l)
        p.prepare_width(F)
        assert_close(run_partial(p, X), want, f"F={F} l={l}")
