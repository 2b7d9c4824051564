"""Rows that are cut into pieces by group boundaries: their sums by a few lanes, by a wavefront and by a
workgroup, at the numbers of pieces where one takes over from the other."""
import numpy as np
import pytest
import torch

import graphgen
import oracle
import paper_2204_02662_amd as epp
from _util import assert_close, dev, run_partial

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("F", [1, 3, 4, 6, 16, 41, 64, 130, 300])
def test_rows_of_every_number_of_pieces(F):
    gs = 8
    lanes = 1
    while lanes * (1 if F < 4 else 4) < F and lanes < 64:
        lanes *= 2
    wide = 64 * 64 // lanes  # more pieces than this: all wavefronts
    pieces = [2, 3, 9, 10, 17, 23, 24, 25, 26, 63, 64, 65, wide - 1, wide, wide + 1, wide + 2, 2 * wide + 37]
    # (between them rows of one entry: the first group of a cut row then starts at any place in it)
    lengths = np.concatenate([[gs * m - 3, 1] for m in pieces])
    n = int(lengths.max()) + 8
    rng = np.random.default_rng(61)
    lens = np.ones(n, np.int64)
    lens[: lengths.size] = lengths
    rowptr = np.zeros(n + 1, np.int32)
    rowptr[1:] = np.cumsum(lens)
    col = np.concatenate([np.sort(rng.choice(n, size=k, replace=False)) for k in lens]).astype(np.int32)
    val = (rng.standard_normal(col.size) / np.sqrt(np.repeat(lens, lens))).astype(np.float32)
    train = np.arange(n, dtype=np.int32)
    sets_o, paths_o = oracle.prepare(n, rowptr, col, val, train, 1)
    paths = epp.epp_prepare(n, *(torch.from_numpy(a).to(dev()) for a in (rowptr, col, val, train)), 1)
    X = graphgen.normal_rows(n, F, sets_o[0], 62)
    p = paths.path(0)
    p.set_group_size(F, gs)
    got = run_partial(p, X)
    assert_close(got, oracle.path_aggregate(n, paths_o[0], X), f"F={F}")
    assert np.array_equal(got, run_partial(p, X))  # equal inputs, equal bits
    assert p.info().n_split_rows >= len(pieces)
