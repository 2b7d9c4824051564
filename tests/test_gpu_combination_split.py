"""Both products where they are taken in bfloat16 parts (two widths of 65 to 128, many rows): edges of the widths and row counts, and
operands that the parts cannot hold."""
import numpy as np
import pytest
import torch

import paper_2204_02662_amd as epp
from _util import dev

pytestmark = pytest.mark.gpu


def _run(m, Fi, Fo, change=lambda Y, G, W, rows: None):
    """(W', Y', their values in 64 bits, the sums of the products' magnitudes) over m vertices of a graph of self-loops."""
    n = m + 50
    rng = np.random.default_rng(m + Fi + Fo)
    rows = np.sort(rng.permutation(n)[:m])
    Y, G, W = (rng.standard_normal(s).astype(np.float32) for s in ((n, Fi), (n, Fo), (Fi, Fo)))
    change(Y, G, W, rows)
    g = (np.arange(n + 1, dtype=np.int32), np.arange(n, dtype=np.int32), np.ones(n, np.float32), rows.astype(np.int32))
    paths = epp.epp_prepare(n, *(torch.from_numpy(a).to(dev()) for a in g), 1)
    Yd, Gd, Wd = (torch.from_numpy(a).to(dev()) for a in (Y, G, W))
    gW, gS, gY = torch.empty(Fi, Fo, device=dev()), torch.empty(Fi, Fo, device=dev()), torch.full((n, Fi), 5.0, device=dev())
    ws = torch.empty(epp.epp_weight_gradient_workspace(paths, 0, Fi, Fo), dtype=torch.uint8, device=dev())
    epp.epp_weight_gradient(paths, 0, Yd, Gd, gW, ws)
    epp.epp_weight_gradient_static(paths, 0, Yd, Gd, gS)
    epp.epp_input_gradient(paths, 0, Gd, Wd, gY)
    assert torch.equal(torch.nan_to_num(gW), torch.nan_to_num(gS))
    got = gY.cpu().numpy()
    outside = np.ones(n, bool)
    outside[rows] = False
    assert np.all(got[outside] == 5.0)
    y, x, w = Y[rows].astype(np.float64), G[rows].astype(np.float64), W.astype(np.float64)
    with np.errstate(invalid="ignore", over="ignore"):
        return gW.cpu().numpy(), got[rows], y.T @ x, x @ w.T, np.abs(y).T @ np.abs(x), np.abs(x) @ np.abs(w).T


def _check(gW, gY, dW, dY, sW, sY):
    # Any order of 32-bit sums: longest chain times 2^-24 of the magnitudes.  Y': 8 + 40 instructions; W': 144 steps of a piece and their 720
    # small products, which are below 2^-8 of the others, then up to 4 pieces.  Never more than at 1e-5, and nothing absolute.
    assert np.all(np.abs(gY - dY) <= 50 * 2.0 ** -24 * sY)
    assert np.all(np.abs(gW - dW) <= 1e-5 * sW)


@pytest.mark.parametrize("Fi,Fo", [(65, 65), (128, 128), (96, 96), (97, 66), (66, 99), (127, 126), (80, 128)])
@pytest.mark.parametrize("m", [16_385, 32_769, 65_537])
def test_widths_and_rows(Fi, Fo, m):
    _check(*_run(m, Fi, Fo))


def test_several_pieces_per_sum():
    _check(*_run(1_300_001, 65, 66))


def _scale(what, factor, where):
    def change(Y, G, W, rows):
        {"Y": Y, "G": G, "W": W}[what][where] *= np.float32(factor)
    return change


@pytest.mark.parametrize("what", ["Y", "G", "W"])
@pytest.mark.parametrize("factor", [2.0 ** -118, 2.0 ** -95, 2.0 ** 60, 2.0 ** 110])
@pytest.mark.parametrize("where", [slice(None), (slice(None), 67), (slice(40, None), slice(None))])
def test_ranges(what, factor, where):
    gW, gY, dW, dY, sW, sY = _run(40_000, 70, 72, _scale(what, factor, where))
    # (results below 2^-126 have fewer bits)
    assert np.all(np.abs(gY - dY) <= 50 * 2.0 ** -24 * sY + 72 * 2.0 ** -149)
    assert np.all(np.abs(gW - dW) <= 1e-5 * sW + 40_000 * 2.0 ** -149)


def test_products_below_the_smallest_normal_number():
    def change(Y, G, W, rows):
        Y *= np.float32(2.0 ** -60)
        G *= np.float32(2.0 ** -70)
        W *= np.float32(2.0 ** -60)
    gW, gY, dW, dY, sW, sY = _run(40_000, 70, 72, change)
    assert np.all(np.abs(gY - dY) <= 50 * 2.0 ** -24 * sY + 72 * 2.0 ** -149)
    assert np.all(np.abs(gW - dW) <= 1e-5 * sW + 40_000 * 2.0 ** -149)


@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan, 3.4e38])
@pytest.mark.parametrize("what", ["Y", "G", "W"])
def test_not_finite(what, value):
    """As in 64 bits: nothing but the rows and columns that have the value is touched by it."""
    def change(Y, G, W, rows):
        if what == "W":
            W[69, 71] = value
        else:
            (Y if what == "Y" else G)[rows[20_003], 66] = value
    gW, gY, dW, dY, sW, sY = _run(40_000, 70, 72, change)
    for got, want, scale in ((gW, dW, sW), (gY, dY, sY)):
        want32 = np.where(np.abs(want) > 3.4028235e38, np.sign(want) * np.inf, want)
        near = np.isfinite(want) & (np.abs(want) > 3e38) | np.isnan(want32)  # (about to overflow: either)
        assert np.array_equal(np.isnan(got) & ~near, np.isnan(want32) & ~near)
        assert np.all(np.isnan(got[np.isnan(want)]))
        whole = np.isfinite(want32) & ~near
        assert np.array_equal(got[np.isinf(want32) & ~near], want32[np.isinf(want32) & ~near])
        assert np.all(np.abs(got[whole] - want[whole]) <= 1e-5 * scale[whole])
