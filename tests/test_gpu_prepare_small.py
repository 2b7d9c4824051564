"""The one-launch construction around the sizes up to which a graph is held in registers."""
import numpy as np
import pytest
import torch

import oracle
import paper_2204_02662_amd as epp
from _util import assert_paths_bit_exact, dev, gpu_prepare

pytestmark = pytest.mark.gpu


class _Random:
    """nnz entries, unevenly spread over the rows (some empty, one long), directed."""

    def __init__(self, n, nnz, seed):
        rng = np.random.default_rng(seed)
        cells = set()
        while len(cells) < nnz:
            row = (n * rng.random(2 * nnz) ** 3).astype(np.int64)
            for c in (row * n + rng.integers(0, n, 2 * nnz)).tolist():
                if len(cells) < nnz:
                    cells.add(c)
        keys = np.sort(np.fromiter(cells, np.int64, nnz))
        self.n, self.col = n, (keys % n).astype(np.int32)
        self.rowptr = np.searchsorted(keys, np.arange(n + 1, dtype=np.int64) * n).astype(np.int32)
        self.val = rng.standard_normal(nnz).astype(np.float32)


@pytest.mark.parametrize("n,nnz", [(1, 1), (1, 0), (63, 200), (64, 4_096), (65, 1), (1_025, 16_383), (4_095, 16_384), (4_096, 16_384),
                                   (4_097, 16_384), (4_096, 16_385), (4_096, 15_361), (130, 16_384)])
def test_around_the_limits(n, nnz):
    g = _Random(n, nnz, n + nnz)
    rng = np.random.default_rng(5)
    for L, m in ((1, 1), (2, max(1, n // 50)), (5, max(1, n // 300)), (3, n)):
        train = np.sort(rng.choice(n, m, replace=False)).astype(np.int32)
        sets_o, paths_o = oracle.prepare(g.n, g.rowptr, g.col, g.val, train, L)
        assert_paths_bit_exact(gpu_prepare(g, train, L), sets_o, paths_o, L)


@pytest.mark.parametrize("where,value", [("col", -1), ("col", 4_000), ("col", 2 ** 31 - 1), ("rowptr", -5), ("rowptr", 16_001),
                                         ("first", 1), ("last", 15_999), ("train", 4_000), ("train", -1)])
def test_mistakes_in_the_input(where, value):
    g = _Random(4_000, 16_000, 9)
    train = np.arange(0, 4_000, 7, dtype=np.int32)
    if where == "col":
        g.col[9_999] = value
    elif where == "train":
        train[100] = value
    else:
        g.rowptr[{"rowptr": 2_000, "first": 0, "last": g.n}[where]] = value
    with pytest.raises(epp.EppError):
        gpu_prepare(g, train, 2)
    torch.cuda.synchronize()


@pytest.mark.parametrize("busy", [0, 60])
@pytest.mark.parametrize("n,nnz", [(3_000, 9_000), (9_000, 40_000), (60_000, 300_000)])
def test_what_has_returned_is_there(n, nnz, busy):
    """Paths made on one stream, behind other work or not, are used on another one as soon as the call is back (no wait in between)."""
    g = _Random(n, nnz, 31)
    train = np.arange(0, n, 5, dtype=np.int32)
    sets_o, paths_o = oracle.prepare(g.n, g.rowptr, g.col, g.val, train, 2)
    arrays = [torch.from_numpy(a).to(dev()) for a in (g.rowptr, g.col, g.val, train)]
    X = torch.randn(n, 8, device=dev(), generator=torch.Generator(dev()).manual_seed(1))
    work = torch.randn(4_096, 4_096, device=dev())
    one, two = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    for _ in range(5):
        with torch.cuda.stream(one):
            for _ in range(busy):
                work = work @ work * 1e-3  # (about a millisecond each)
            paths = epp.epp_prepare(n, *arrays, 2)
            saved = [paths.path(l).export() for l in range(2)]
            again = epp.epp_paths_import(n, arrays[3], saved)
            for p in (paths, again):
                p.path(0).prepare_width(8)
        with torch.cuda.stream(two):
            out = [torch.zeros_like(X) for _ in range(2)]
            for p, o in zip((paths, again), out):
                epp.epp_backward_aggregate(p.path(0), X, o)
        torch.cuda.synchronize()
        want = oracle.path_aggregate(n, paths_o[0], np.where(sets_o[1][:, None] != 0, X.cpu().numpy(), 0))
        for o in out:
            # (sums of at most 300 products of normal numbers in any order)
            assert np.all(np.abs(o.cpu().numpy() - want) <= 1e-4 + 1e-5 * np.abs(want))
