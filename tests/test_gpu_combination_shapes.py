"""Both products of the combination stage at the row counts where the cutting of the rows changes, for every
arrangement of 32-wide blocks, widths that their loads do not divide among them."""
import numpy as np
import pytest
import torch

import graphgen
import oracle
import paper_2204_02662_amd as epp
from _util import dev

pytestmark = pytest.mark.gpu

# (blocks of the first width) x (blocks of the second), widths that are multiples of the load and that are not
SHAPES = [(1, 1), (3, 5), (33, 31), (16, 41), (16, 49), (32, 64), (7, 128), (41, 41), (64, 62), (39, 96), (64, 97), (96, 39),
          (126, 64), (100, 5), (65, 65), (96, 96), (127, 128), (128, 126), (128, 128)]


def _products(n, rows, Fi, Fo, seed):
    """Weight and input gradient over the training set `rows` of a graph of n vertices with self-loops only."""
    rng = np.random.default_rng(seed)
    loops = np.arange(n, dtype=np.int32)
    g = (np.arange(n + 1, dtype=np.int32), loops, np.ones(n, np.float32), rows.astype(np.int32))
    paths = epp.epp_prepare(n, *(torch.from_numpy(a).to(dev()) for a in g), 1)
    Y, W = (rng.standard_normal(s).astype(np.float32) for s in ((n, Fi), (Fi, Fo)))
    G = np.full((n, Fo), np.nan, np.float32)  # rows outside the set are never read
    G[rows] = rng.standard_normal((rows.size, Fo)).astype(np.float32)
    Yd, Gd, Wd = (torch.from_numpy(a).to(dev()) for a in (Y, G, W))
    gW, gS, gY = torch.empty(Fi, Fo, device=dev()), torch.empty(Fi, Fo, device=dev()), torch.full((n, Fi), 5.0, device=dev())
    ws = torch.empty(epp.epp_weight_gradient_workspace(paths, 0, Fi, Fo), dtype=torch.uint8, device=dev())
    epp.epp_weight_gradient(paths, 0, Yd, Gd, gW, ws)
    epp.epp_weight_gradient_static(paths, 0, Yd, Gd, gS)
    epp.epp_input_gradient(paths, 0, Gd, Wd, gY)
    assert torch.equal(gW, gS)
    member = np.zeros(n, np.uint8)
    member[rows] = 1
    G0 = np.where(member[:, None] != 0, G, 0)
    want, scale = oracle.weight_gradient(Y, G0, member)
    assert np.all(np.abs(gW.cpu().numpy() - want) <= 1e-6 + 1e-5 * scale)
    got = gY.cpu().numpy()
    assert np.all(got[member == 0] == 5.0)
    wide, sc = G[rows].astype(np.float64) @ W.T.astype(np.float64), np.abs(G[rows]).astype(np.float64) @ np.abs(W.T)
    assert np.all(np.abs(got[rows] - wide) <= 1e-6 + 1e-5 * sc)


@pytest.mark.parametrize("Fi,Fo", SHAPES)
def test_few_rows(Fi, Fo):
    n = 3_000
    order = np.random.default_rng(71).permutation(n)
    for m in (1, 2, 7, 17, 63, 64, 65, 256, 257, 1_025, 2_999):
        _products(n, np.sort(order[:m]), Fi, Fo, m)


@pytest.mark.parametrize("m", [16_383, 32_769, 49_999, 50_001, 65_536, 65_537])
@pytest.mark.parametrize("Fi,Fo", [(16, 16), (16, 64), (5, 128), (64, 64), (39, 96), (96, 96)])
def test_many_rows(Fi, Fo, m):
    _products(70_000, np.sort(np.random.default_rng(72).permutation(70_000)[:m]), Fi, Fo, m)
