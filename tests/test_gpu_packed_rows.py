"""Source rows of widths that lie across the ends of 128-byte lines: copied to a wider stride by the launch,
or read 16 bytes a lane where they are, the last lane ending at the row's end."""
import numpy as np
import pytest
import torch

import graphgen
import oracle
import paper_2204_02662_amd as epp
from _util import assert_close, dev, gpu_prepare, gpu_prepare_full, run_full, run_partial

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("layout", ["plain", "partitioned", "shared"])
@pytest.mark.parametrize("packed", ["2", "0"])
@pytest.mark.parametrize("F", [5, 7, 15, 17, 31, 33, 47, 63, 65, 127, 129, 259])
def test_rows_of_odd_width(F, packed, layout, monkeypatch):
    monkeypatch.setenv("EPP_TUNE_ROWS", "0")
    monkeypatch.setenv("EPP_TUNE_PACK", packed)
    monkeypatch.setenv("EPP_TUNE_SHARE_PCT", "1" if layout == "shared" else "0")
    monkeypatch.setenv("EPP_TUNE_PART", "2" if layout == "partitioned" else "0")
    monkeypatch.setenv("EPP_TUNE_PART_KB", "16")
    monkeypatch.setenv("EPP_TUNE_PART_MINLEN", "8")
    g = graphgen.random_graph("rmat", 5_003, seed=471, raw_draws=60_000)  # (the last word of a bitmap is not full)
    train = graphgen.training_set(g.n, 700, 472)
    sets_o, paths_o = oracle.prepare(g.n, g.rowptr, g.col, g.val, train, 2)
    monkeypatch.setenv("EPP_TUNE_SMALL_PREPARE", "0")
    paths = gpu_prepare(g, train, 2)
    for l in (1, 0):
        src, rows = sets_o[1 - l].astype(bool), sets_o[2 - l].astype(bool)
        X = graphgen.normal_rows(g.n, F, sets_o[1 - l], 473 + l)
        want = oracle.path_aggregate(g.n, paths_o[l], X)
        X[~src] = np.nan  # never read, packed or not
        p = paths.path(l)
        p.set_group_size(F, 24)
        got = run_partial(p, X, poison=9.0)
        assert np.all(got[~rows] == 9.0)
        assert_close(got[rows], want[rows], f"F={F} l={l}")
        assert np.array_equal(got[rows], run_partial(p, X, poison=1.0)[rows])
    assert (paths.path(0).info().part_rows > 0) == (layout == "partitioned")
    full = gpu_prepare_full(g)
    X = graphgen.normal_rows(g.n, F, None, 479)
    assert_close(run_full(full, X), oracle.full_aggregate(g.n, g.rowptr, g.col, g.val, X), f"all-active F={F}")


def test_captured_launch_packs_the_rows_of_each_replay(monkeypatch):
    monkeypatch.setenv("EPP_TUNE_ROWS", "0")
    monkeypatch.setenv("EPP_TUNE_PACK", "2")
    g = graphgen.random_graph("rmat", 5_003, seed=471, raw_draws=60_000)
    full = gpu_prepare_full(g)
    full.prepare_width(47)
    x = torch.zeros(g.n, 47, device=dev())
    y = torch.empty_like(x)
    epp.epp_full_aggregate(full, x, y)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        epp.epp_full_aggregate(full, x, y)
    for rep in range(3):
        x.normal_()
        graph.replay()
        torch.cuda.synchronize()
        z = torch.empty_like(y)
        epp.epp_full_aggregate(full, x, z)
        assert torch.equal(y, z), f"replay {rep}"
        assert_close(y.cpu().numpy(), oracle.full_aggregate(g.n, g.rowptr, g.col, g.val, x.cpu().numpy()), f"replay {rep}")
