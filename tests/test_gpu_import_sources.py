"""Imported paths whose columns are not all in the source set that the training ids and the next path name: the
launch gathers the caller's rows all the same, also where it first copies the source rows."""
import numpy as np
import pytest
import torch

import graphgen
import oracle
import paper_2204_02662_amd as epp
from _util import assert_close, dev, gpu_prepare, run_partial

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("packed", ["0", "2"])
@pytest.mark.parametrize("F", [7, 17, 47])
def test_columns_outside_the_source_set(F, packed, monkeypatch):
    monkeypatch.setenv("EPP_TUNE_ROWS", "0")
    monkeypatch.setenv("EPP_TUNE_PACK", packed)
    g = graphgen.random_graph("rmat", 3_001, seed=81, raw_draws=30_000)
    train = graphgen.training_set(g.n, 400, 82)
    sets_o, paths_o = oracle.prepare(g.n, g.rowptr, g.col, g.val, train, 2)
    saved = [gpu_prepare(g, train, 2).path(l).export() for l in range(2)]
    X = graphgen.normal_rows(g.n, F, sets_o[0], 83)
    want = oracle.path_aggregate(g.n, paths_o[1], X)
    stale = torch.full((4 << 20,), float("nan"), device=dev())  # what the library may be given next
    del stale
    for ids in (train, train[:100]):  # the saved training set, and another one
        paths = epp.epp_paths_import(g.n, torch.from_numpy(np.ascontiguousarray(ids, np.int32)).to(dev()), saved)
        p = paths.path(1)
        p.prepare_width(F)
        assert_close(run_partial(p, X), want, f"F={F} {ids.size} training ids")
