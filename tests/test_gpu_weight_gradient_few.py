"""Weight gradients of few rows, which one launch forms, at the ends of the wavefronts' shares, of the 32 x 32 blocks and of the rule."""
import numpy as np
import pytest
import torch

import paper_2204_02662_amd as epp
from _util import dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Fi,Fo", [(1, 1), (3, 33), (32, 32), (41, 64), (100, 7), (128, 128)])
@pytest.mark.parametrize("rows", [1, 2, 3, 16, 31, 32, 33, 95, 383, 384, 385])
def test_edges(rows, Fi, Fo):
    n, rng = 1_000, np.random.default_rng(rows * 1000 + Fi + Fo)
    gen = torch.Generator(dev()).manual_seed(rows)
    ids = torch.from_numpy(np.sort(rng.choice(n, size=rows, replace=False)).astype(np.int32)).to(dev())
    eye = [torch.arange(n + 1, dtype=torch.int32, device=dev()), torch.arange(n, dtype=torch.int32, device=dev()), torch.ones(n, device=dev())]
    paths = epp.epp_prepare(n, *eye, ids, 1)
    every = epp.epp_prepare(rows, eye[0][:rows + 1], eye[1][:rows], eye[2][:rows], eye[1][:rows], 1)  # (k = -1: no ids)
    Y, X = torch.randn(n, Fi, device=dev(), generator=gen), torch.randn(n, Fo, device=dev(), generator=gen)
    outside = torch.ones(n, dtype=torch.bool, device=dev())
    outside[ids.long()] = False
    Y[outside], X[outside] = float("nan"), float("inf")  # (no row but the set's counts)
    y, x = Y[ids.long()], X[ids.long()]
    want, size = y.double().T @ x.double(), y.double().abs().T @ x.double().abs()
    for handle, k, a, b in ((paths, 0, Y, X), (every, -1, y, x)):
        ws = torch.empty(epp.epp_weight_gradient_workspace(handle, k, Fi, Fo), dtype=torch.uint8, device=dev())
        got, again = (torch.full((Fi, Fo), float("nan"), device=dev()) for _ in range(2))
        epp.epp_weight_gradient(handle, k, a, b, got, ws)
        epp.epp_weight_gradient_static(handle, k, a, b, again)
        # 16 rows to a chain at most, two additions of chains, a rounding: 20 roundings of 2^-24 of the terms' sizes
        assert torch.all((got.double() - want).abs() <= 20 * 2.0 ** -24 * size), (got.double() - want).abs().max()
        assert torch.equal(got, again)
    # the last row twice, the second time with nothing: an infinity stays one
    if rows % 2:
        Y[ids[-1].long(), 0] = float("inf")
        epp.epp_weight_gradient_static(paths, 0, Y, X, got)
        assert torch.equal(got[0], torch.where(X[ids[-1].long()] > 0, float("inf"), float("-inf")))
        assert torch.isfinite(got[1:]).all()


@pytest.mark.parametrize("Fi,Fo", [(5, 4), (41, 64), (128, 128), (129, 16)])
def test_workspace(Fi, Fo):
    """One block of W', the least there is, where no partial sums are formed; as many as the rows make beyond, and at other widths."""
    for rows in (0, 1, 60, 256, 384, 385, 2_000):
        eye = torch.arange(2_001, dtype=torch.int32, device=dev())
        paths = epp.epp_prepare(2_000, eye, eye[:2_000].clone(), torch.ones(2_000, device=dev()), eye[:rows].clone(), 1)
        blocks, rest = divmod(epp.epp_weight_gradient_workspace(paths, 0, Fi, Fo), Fi * Fo * 4)
        assert rest == 0 and (blocks == 1 if rows <= 384 and max(Fi, Fo) <= 128 else blocks >= 1), rows
        if rows >= 385 and max(Fi, Fo) <= 128:
            assert blocks == -(-rows // 64)
        Y, X = torch.ones(2_000, Fi, device=dev()), torch.ones(2_000, Fo, device=dev())
        need = blocks * Fi * Fo * 4
        held = torch.full((need + 256,), 7, dtype=torch.uint8, device=dev())
        got = torch.empty(Fi, Fo, device=dev())
        epp.epp_weight_gradient(paths, 0, Y, X, got, held[:need])
        assert torch.all(got == rows) and torch.all(held[need:] == 7), rows
        with pytest.raises(epp.EppError):
            epp.epp_weight_gradient(paths, 0, Y, X, got, held[:need - 16])
