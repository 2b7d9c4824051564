"""Products in bfloat16 parts: what each of the parts is there for, small operands beside large ones that meet zeros, and what is formed
again in fp32 in one piece of a workgroup's rows only."""
import numpy as np
import pytest
import torch

import paper_2204_02662_amd as epp
from _util import dev
from test_gpu_combination_split import _run

pytestmark = pytest.mark.gpu
U = 2.0 ** -24
TINY = 2.0 ** -149


@pytest.mark.parametrize("Fi,Fo", [(65, 66), (128, 128), (97, 80)])
@pytest.mark.parametrize("scale", [1.0, 2.0 ** -110, 2.0 ** 30])
def test_sums_of_one_product(Fi, Fo, scale):
    def change(Y, G, W, rows):
        rng = np.random.default_rng(Fi)
        keep = rows[rng.permutation(rows.size)[:Fo]]
        values = G[keep, np.arange(Fo)] * np.float32(scale)
        G[:] = 0
        G[keep, np.arange(Fo)] = values
    gW, gY, dW, dY, _, _ = _run(40_000, Fi, Fo, change)
    # Left out: at most 2 x 2^-8 x 2^-17 (and 2^-34) of the product.  Rounded: the small products' sum (of 2^-6.4 at most, five times by
    # 2^-23) and the whole, once.
    assert np.all(np.abs(gY - dY) <= (1 + 1 + 0.2) * U * np.abs(dY) + TINY)
    assert np.all(np.abs(gW - dW) <= (1 + 1 + 0.2) * U * np.abs(dW) + TINY)


@pytest.mark.parametrize("Fi,Fo", [(65, 67), (96, 96), (128, 128)])
def test_two_chains(Fi, Fo):
    """Errors of sums of normal numbers, over all of them: half of what the fp32 instruction has (1.3 to 2.0e-7), less than with the small
    products in the chain of the large ones (1.6e-7 for Y', 2.4e-7 for W'), far less than without the third parts (3e-6)."""
    gW, gY, dW, dY, _, _ = _run(70_000, Fi, Fo)
    assert np.linalg.norm(gY - dY) <= 0.9e-7 * np.linalg.norm(dY)
    assert np.linalg.norm(gW - dW) <= 1.25e-7 * np.linalg.norm(dW)


@pytest.mark.parametrize("exponent", [-90, -105, -118, -126, -140])
def test_small_operands_beside_one_that_meets_a_zero(exponent):
    small = np.float32(2.0 ** exponent)

    def change(Y, G, W, rows):
        for x in (Y, G, W):
            x[:] = np.abs(x) + 1
        Y *= small
        Y[rows[20_001]] = 1
        G[rows[20_001]] = 0  # W'
        G[rows[30_000:]] *= small
        G[rows[30_000:], 7] = 1
        W[:, 7] = 0          # Y' of these rows
        G[rows[:30_000], 7] = 0
    gW, gY, dW, dY, sW, sY = _run(40_000, 70, 72, change)
    assert np.all(np.abs(gY - dY) <= 50 * U * sY + 72 * TINY)
    # (all of one sign: a part of 160 rows is at most 20 roundings off, and 500 such parts are added in 64 bits, half of which
    # products are those of two small numbers)
    assert np.all(np.abs(gW - dW) <= 22 * U * sW + 500 * TINY)


@pytest.mark.parametrize("at", [100, 2_304 + 100])
@pytest.mark.parametrize("what,value", [("Y", np.inf), ("G", 2.0 ** 110), ("Y", 2.0 ** -118), ("G", np.nan)])
def test_one_piece_of_several(what, value, at):
    """1.3 M rows: 2,544 a workgroup, in pieces of 2,304 and 240."""
    def change(Y, G, W, rows):
        (Y if what == "Y" else G)[rows[at], 64] = value
    gW, gY, dW, dY, sW, sY = _run(1_300_001, 65, 66, change)
    for got, want, scale in ((gW, dW, sW), (gY, dY, sY)):
        whole = np.isfinite(want)
        assert np.array_equal(np.isnan(got), np.isnan(want))
        assert np.array_equal(got[np.isinf(want)], want[np.isinf(want)].astype(np.float32))
        assert np.all(np.abs(got[whole] - want[whole]) <= 1e-5 * scale[whole])
    if what == "Y":  # the rows that are not 64 of W' have nothing to do with it
        assert np.linalg.norm(gW[:64] - dW[:64]) <= 4e-7 * np.linalg.norm(dW[:64])


@pytest.mark.parametrize("n", [32_769, 40_001])
def test_all_vertices(n):
    gen = torch.Generator(dev()).manual_seed(n)
    G, W = (torch.randn(*s, device=dev(), generator=gen) for s in ((n, 67), (66, 67)))
    ids = torch.arange(n, dtype=torch.int32, device=dev())
    paths = epp.epp_prepare(n, torch.arange(n + 1, dtype=torch.int32, device=dev()), ids, torch.ones(n, device=dev()), ids[:7].clone(), 1)
    got = torch.full((n, 66), 5.0, device=dev())
    epp.epp_input_gradient(paths, -1, G, W, got)
    x, w = G.cpu().numpy().astype(np.float64), W.cpu().numpy().astype(np.float64)
    assert np.all(np.abs(got.cpu().numpy() - x @ w.T) <= 50 * U * (np.abs(x) @ np.abs(w).T))
