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


@pytest.mark.parametrize("nnz,log2", [(3_030_303, 9), (3_030_304, 10), (5_882_352, 10), (5_882_353, 11)])
def test_lists_of_paths_by_their_entries(nnz, log2, monkeypatch):
    """Either side of the two numbers of entries from which on a path's list begins with longer rows: the widths whose chunks it goes down to
    take it, the others make one of their own, and both give what the oracle does."""
    for k, v in {"ROWS": 2, "SMALL_PREPARE": 0}.items():
        monkeypatch.setenv("EPP_TUNE_" + k, str(v))
    rng = np.random.default_rng(nnz)
    n = 200_003  # (a prime: multiples of a stride below it, as many as a row has, are different columns)
    lens = np.ones(n, np.int64)
    lens[rng.permutation(n)[:len(EDGES) * 8]] = EDGES * 8
    spare = np.flatnonzero(lens == 1)
    lens[spare] += (nnz - lens.sum()) // spare.size
    lens[spare[:nnz - lens.sum()]] += 1
    rowptr = np.zeros(n + 1, np.int64)
    rowptr[1:] = np.cumsum(lens)
    row = np.repeat(np.arange(n), lens)
    col = ((rng.integers(0, n, size=n)[row] + (np.arange(nnz) - rowptr[row]) * rng.integers(1, n, size=n)[row]) % n).astype(np.int32)
    val = (rng.standard_normal(nnz) / np.sqrt(np.repeat(lens, lens))).astype(np.float32)
    rowptr, train = rowptr.astype(np.int32), np.arange(n, dtype=np.int32)
    sets_o, paths_o = oracle.prepare(n, rowptr, col, val, train, 1)
    ids = torch.from_numpy(train).to(dev())
    prepared = epp.epp_prepare(n, *(torch.from_numpy(a).to(dev()) for a in (rowptr, col, val)), ids, 1)
    imported = epp.epp_paths_import(n, ids, [prepared.path(0).export()])
    for F, chunk_log2 in ((16, 11), (24, 10), (41, 9)):
        X = graphgen.normal_rows(n, F, sets_o[0], 3)
        want, x, first = oracle.path_aggregate(n, paths_o[0], X), torch.from_numpy(X).to(dev()), None
        for what, paths in (("prepared", prepared), ("imported", imported)):
            p = paths.path(0)
            i = p.info()
            assert i.nnz == nnz
            p.prepare_width(F)
            sums = sum(rows << (c - chunk_log2) for c, rows in enumerate(i.len_hist) if c > chunk_log2) * F * 4
            assert (p.info().bytes - i.bytes == sums) == (log2 <= chunk_log2), f"F={F} {what}"
            for _ in range(2):
                out = torch.full((n, F), float("nan"), device=dev())
                epp.epp_backward_aggregate(p, x, out)
                if first is None:
                    assert_close(out.cpu().numpy(), want, f"F={F} {what}")
                    first = out
                assert torch.equal(out, first), f"F={F} {what}"
