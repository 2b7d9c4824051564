"""Long rows of the row kernel, which a construction and an import list class by class beside the path: every route to such a list, rows at
the edges of the classes, more of them in a workgroup than one, and none."""
import numpy as np
import pytest
import torch

import graphgen
import oracle
import paper_2204_02662_amd as epp
from _util import assert_close, dev

pytestmark = pytest.mark.gpu

EDGES = [511, 512, 513, 1023, 1024, 1025, 2047, 2048, 2049, 4096, 4097, 8192, 8193, 9000]


@pytest.mark.parametrize("F", [4, 16, 41])  # chunks of 8192, 2048 and 512 entries
@pytest.mark.parametrize("lengths", [EDGES, [700] * 600, [513, 1030, 2100] * 90, [512] * 40], ids=["edges", "all", "classes", "none"])
def test_every_route(lengths, F, monkeypatch):
    monkeypatch.setenv("EPP_TUNE_ROWS", "2")
    rng = np.random.default_rng(7)
    n = max(10_000, len(lengths))
    lens = np.ones(n, np.int64)
    # (beside each other, as well as far apart: several rows of a workgroup's 256)
    at = np.concatenate([np.arange(len(lengths) // 2), rng.permutation(np.arange(len(lengths), n))[:len(lengths) - len(lengths) // 2]])
    lens[at] = lengths
    rowptr = np.zeros(n + 1, np.int32)
    rowptr[1:] = np.cumsum(lens)
    col = np.concatenate([np.sort(rng.choice(n, size=k, replace=False)) for k in lens]).astype(np.int32)
    val = (rng.standard_normal(col.size) / np.sqrt(np.repeat(lens, lens))).astype(np.float32)
    train = np.arange(n, dtype=np.int32)
    sets_o, paths_o = oracle.prepare(n, rowptr, col, val, train, 1)
    X = graphgen.normal_rows(n, F, sets_o[0], 3)
    want = oracle.path_aggregate(n, paths_o[0], X)
    csr = [torch.from_numpy(a).to(dev()) for a in (rowptr, col, val)]
    ids, x = torch.from_numpy(train).to(dev()), torch.from_numpy(X).to(dev())
    built = {}
    for small in "01":  # (small graphs: one launch, which lists nothing)
        monkeypatch.setenv("EPP_TUNE_SMALL_PREPARE", small)
        built["prepare " + small] = epp.epp_prepare(n, *csr, ids, 1)
    built["import"] = epp.epp_paths_import(n, ids, [built["prepare 0"].path(0).export()])
    first = None
    for what, paths in built.items():
        p = paths.path(0)
        for width in (F, F, 70):  # (another width's chunks, 256 entries, have a list of their own)
            p.prepare_width(width)
        for _ in range(2):
            out = torch.full((n, F), float("nan"), device=dev())
            epp.epp_backward_aggregate(p, x, out)
            if first is None:
                assert_close(out.cpu().numpy(), want, f"F={F} {what}")
                first = out
            assert torch.equal(out, first), what
        wide = torch.full((n, 70), float("nan"), device=dev())
        epp.epp_backward_aggregate(p, x[:, torch.arange(70, device=dev()) % F].contiguous(), wide)
        assert_close(wide.cpu().numpy(), want[:, np.arange(70) % F], f"70 floats, {what}")
