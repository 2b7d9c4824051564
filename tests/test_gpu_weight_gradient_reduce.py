"""The sums of the weight gradient's partial sums: either side of every line between the kernels that form them."""
import numpy as np
import pytest
import torch

import paper_2204_02662_amd as epp
from _util import dev

pytestmark = pytest.mark.gpu


# 8,192 / 8,193 rows are 128 / 129 partial sums of two widths of which one is above 32 (32,768 / 32,769 of 16 x 16)
@pytest.mark.parametrize("n,Fi,Fo", [(n, Fi, Fo) for n in (8_192, 8_193, 40_001) for Fi, Fo in (
    (33, 31), (32, 33), (64, 17), (63, 65), (64, 64), (91, 90), (128, 64), (117, 71))] + [
    (32_768, 16, 16), (32_769, 16, 16), (33_000, 5, 1), (70_000, 1, 3), (70_000, 130, 64)])
def test_partial_sums(n, Fi, Fo):
    gen = torch.Generator(dev()).manual_seed(n + Fi + Fo)
    Y, G = (torch.randn(n, F, device=dev(), generator=gen) for F in (Fi, Fo))
    ids = torch.arange(n, dtype=torch.int32, device=dev())
    paths = epp.epp_prepare(n, torch.arange(n + 1, dtype=torch.int32, device=dev()), ids, torch.ones(n, device=dev()), ids[:7].clone(), 1)
    got, again = torch.full((Fi, Fo), 5.0, device=dev()), torch.empty(Fi, Fo, device=dev())
    ws = torch.empty(epp.epp_weight_gradient_workspace(paths, -1, Fi, Fo), dtype=torch.uint8, device=dev())
    epp.epp_weight_gradient(paths, -1, Y, G, got, ws)
    epp.epp_weight_gradient(paths, -1, Y, G, again, ws)
    assert torch.equal(got, again)
    y, x = Y.cpu().numpy().astype(np.float64), G.cpu().numpy().astype(np.float64)
    # (32-bit sums of at most 256 rows in a chain, the rest in 64 bits)
    assert np.all(np.abs(got.cpu().numpy() - y.T @ x) <= 1e-5 * (np.abs(y).T @ np.abs(x)))
