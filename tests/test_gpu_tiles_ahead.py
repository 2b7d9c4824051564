"""How far a launch on tiles gathers ahead, and how it addresses its source rows, changes no bit of what it gives."""
import numpy as np
import pytest
import torch

import graphgen
import oracle
import paper_2204_02662_amd as epp
from _util import assert_close, dev, gpu_prepare

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lanes,aheads", [(4, (4,)), (8, (2, 3, 4)), (16, (0, 3))])
@pytest.mark.parametrize("F", [6, 33, 64, 100])
def test_windows_and_addresses(lanes, aheads, F, monkeypatch):
    """The outer path and the inner one on its tiles, whose other sources hold NaN; rows that begin at 4 bytes of 16."""
    for k, v in {"ROWS": 0, "TILES": 2, "TILE_LANES": lanes, "TILES_AT_ONCE": 512, "SMALL_PREPARE": 0, "SHARE_PCT": 1}.items():
        monkeypatch.setenv("EPP_TUNE_" + k, str(v))
    g = graphgen.random_graph("rmat", 60_001, seed=171, raw_draws=500_000)
    train = graphgen.training_set(g.n, 6_000, 172)
    sets_o, paths_o = oracle.prepare(g.n, g.rowptr, g.col, g.val, train, 2)
    for l in (1, 0):
        X = graphgen.normal_rows(g.n, F, sets_o[1 - l], 173 + l)
        want = oracle.path_aggregate(g.n, paths_o[l], X)
        X[~sets_o[1 - l].astype(bool)] = np.nan
        first = None
        for ahead in aheads:
            for far in (0, 1):
                monkeypatch.setenv("EPP_TUNE_TILE_AHEAD", str(ahead))
                monkeypatch.setenv("EPP_TUNE_TILE_FAR", str(far))
                p = gpu_prepare(g, train, 2).path(l)
                p.prepare_width(F)
                for shift in (0, 1):
                    held = torch.empty(g.n * F + 1, device=dev())
                    x = held[shift:shift + g.n * F].view(g.n, F)
                    x.copy_(torch.from_numpy(X))
                    out = torch.full((g.n, F), 9.0, device=dev())
                    epp.epp_backward_aggregate(p, x, out)
                    got = out.cpu().numpy()
                    what = f"lanes={lanes} F={F} l={l} ahead={ahead} far={far} shift={shift}"
                    rows = sets_o[2 - l].astype(bool)
                    assert np.all(got[~rows] == 9.0), what
                    assert_close(got[rows], want[rows], what)
                    first = got if first is None else first
                    assert np.array_equal(got, first), what


@pytest.mark.parametrize("lanes,aheads", [(4, (-1, 0, 2, 3, 5, 196)), (8, (-1, 0, 1, 5, 128, 131)), (16, (-1, 1, 2, 4, 8))])
def test_windows_that_do_not_exist(lanes, aheads, monkeypatch):
    """A switch that asks for one leaves the choice as it is: a launch never runs a kernel made for other lanes than its plan's."""
    for k, v in {"ROWS": 0, "TILES": 2, "TILE_LANES": lanes, "TILES_AT_ONCE": 512, "SMALL_PREPARE": 0}.items():
        monkeypatch.setenv("EPP_TUNE_" + k, str(v))
    g = graphgen.random_graph("rmat", 60_001, seed=171, raw_draws=500_000)
    train, F = graphgen.training_set(g.n, 6_000, 172), 33
    sets_o, paths_o = oracle.prepare(g.n, g.rowptr, g.col, g.val, train, 1)
    X = graphgen.normal_rows(g.n, F, sets_o[0], 175)
    want = oracle.path_aggregate(g.n, paths_o[0], X)
    for ahead in aheads:
        monkeypatch.setenv("EPP_TUNE_TILE_AHEAD", str(ahead))
        p = gpu_prepare(g, train, 1).path(0)
        p.prepare_width(F)
        out = torch.zeros(g.n, F, device=dev())
        epp.epp_backward_aggregate(p, torch.from_numpy(X).to(dev()), out)
        assert_close(out.cpu().numpy(), want, f"lanes={lanes} ahead={ahead}")
