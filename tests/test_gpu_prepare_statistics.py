"""What the kernels of a preparation and of an import hand on beside the paths (sizes, row-length statistics), at the sizes where they are
cleared, counted and handed over in another way: paths per launch of an import, rows per workgroup, tiles per workgroup, training sets of one workgroup."""
import numpy as np
import pytest
import torch

import oracle
import paper_2204_02662_amd as epp
from _util import assert_paths_bit_exact, dev, gpu_prepare
from test_gpu_prepare_levels import _Ring

pytestmark = pytest.mark.gpu


class _Graph:
    def __init__(self, n, nnz, seed):
        rng = np.random.default_rng(seed)
        lens = np.full(n, nnz // n, np.int64)
        lens[: nnz - int(lens.sum())] += 1
        self.n = n
        self.rowptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
        # ascending and distinct: a stride that goes once round the ids at most
        step = n // (int(lens.max()) + 1)
        self.col = np.concatenate([np.sort((rng.integers(n) + step * np.arange(k)) % n) for k in lens]).astype(np.int32)
        self.val = rng.standard_normal(nnz).astype(np.float32)


@pytest.mark.parametrize("L", [1, 3, 4, 5, 9])
def test_imports_of_several_launches(L, monkeypatch):
    monkeypatch.setenv("EPP_TUNE_SMALL_PREPARE", "0")
    g = _Ring(20_011, True, 31)
    train = np.sort(np.random.default_rng(32).choice(g.n, 40, replace=False)).astype(np.int32)
    sets_o, paths_o = oracle.prepare(g.n, g.rowptr, g.col, g.val, train, L)
    paths = gpu_prepare(g, train, L)
    assert_paths_bit_exact(paths, sets_o, paths_o, L)
    saved = [paths.path(l).export() for l in range(L)]
    again = epp.epp_paths_import(g.n, torch.from_numpy(train).to(dev()), saved)
    assert_paths_bit_exact(again, sets_o, paths_o, L)


# vertices: a row's workgroup takes one and several turns; training sets: one workgroup's and more, ids and vertices, none
@pytest.mark.parametrize("n,m", [(20_011, 0), (65_000, 1), (262_144, 65_000), (300_000, 65_537), (524_288, 300), (524_289, 300), (1_100_000, 900)])
def test_sizes_of_sets_and_training_sets(n, m, monkeypatch):
    monkeypatch.setenv("EPP_TUNE_SMALL_PREPARE", "0")
    g = _Ring(n, True, 33)
    train = np.random.default_rng(34).choice(n, m, replace=False).astype(np.int32)
    for _ in range(2):  # (memory that was used before)
        sets_o, paths_o = oracle.prepare(g.n, g.rowptr, g.col, g.val, train, 2)
        paths = gpu_prepare(g, train, 2)
        assert_paths_bit_exact(paths, sets_o, paths_o, 2)
        saved = [paths.path(l).export() for l in range(2)]
        assert_paths_bit_exact(epp.epp_paths_import(n, torch.from_numpy(train).to(dev()), saved), sets_o, paths_o, 2)


@pytest.mark.parametrize("nnz", [2048 * 4, 2048 * 4 + 1, 2048 * 2048, 2048 * 2048 + 1])
def test_tiles_per_workgroup(nnz, monkeypatch):
    monkeypatch.setenv("EPP_TUNE_SMALL_PREPARE", "0")
    g = _Graph(min(60_000, nnz // 3), nnz, 35)
    train = np.random.default_rng(36).choice(g.n, g.n // 100, replace=False).astype(np.int32)
    sets_o, paths_o = oracle.prepare(g.n, g.rowptr, g.col, g.val, train, 2)
    assert_paths_bit_exact(gpu_prepare(g, train, 2), sets_o, paths_o, 2)
