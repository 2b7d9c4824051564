"""Launches of the row kernel for different widths of one path, or for a path and the inner one on its arrays, share nothing that they write:
the chunks of a cut row are counted width by width, also where more widths than the path's list has counts for are in use."""
import numpy as np
import pytest
import torch

import graphgen
import oracle
import paper_2204_02662_amd as epp
from _util import assert_close, dev

pytestmark = pytest.mark.gpu

WIDTHS = [16, 41, 8, 64, 24, 12, 33, 4]  # chunks of 2048, 512, 4096, 512, 1024, 2048, 512 and 8192 entries; five have a count in the list


@pytest.fixture(scope="module")
def graph():
    """40,000 vertices with self-loops, 40 rows of 9,000 to 30,000 entries; half of the vertices train."""
    n, rng = 40_000, np.random.default_rng(31)
    lens = rng.integers(2, 7, size=n)
    lens[rng.permutation(n)[:40]] = rng.integers(9_000, 30_000, size=40)
    rows = [np.union1d(rng.choice(n, size=k, replace=False), [v]).astype(np.int32) for v, k in enumerate(lens)]
    rowptr = np.zeros(n + 1, np.int32)
    rowptr[1:] = np.cumsum([r.size for r in rows])
    col = np.concatenate(rows)
    val = (rng.standard_normal(col.size) / np.sqrt(np.repeat(np.diff(rowptr), np.diff(rowptr)))).astype(np.float32)
    train = np.sort(rng.permutation(n)[:n // 2]).astype(np.int32)
    return n, rowptr, col, val, train, oracle.prepare(n, rowptr, col, val, train, 2)


@pytest.mark.parametrize("route,inner", [("prepared", False), ("imported", False), ("prepared", True)])
def test_widths_side_by_side(route, inner, graph, monkeypatch):
    for k, v in {"ROWS": 2, "SMALL_PREPARE": 0, "SHARE_PCT": 1 if inner else 0}.items():
        monkeypatch.setenv("EPP_TUNE_" + k, str(v))
    n, rowptr, col, val, train, (sets_o, paths_o) = graph
    ids = torch.from_numpy(train).to(dev())
    paths = epp.epp_prepare(n, *(torch.from_numpy(a).to(dev()) for a in (rowptr, col, val)), ids, 2)
    if route == "imported":
        paths = epp.epp_paths_import(n, ids, [paths.path(l).export() for l in range(2)])
    layer = {F: 1 if inner and i % 2 == 0 else 0 for i, F in enumerate(WIDTHS)}
    assert paths.path(1).info().shares_entries == int(inner)
    work, first = {}, {}
    for F in WIDTHS:  # (all prepared before the first launch: the list's counts are dealt out)
        paths.path(layer[F]).prepare_width(F)
    for F in WIDTHS:
        l = layer[F]
        X = graphgen.normal_rows(n, F, sets_o[1 - l], 32 + F)
        work[F] = paths.path(l), torch.from_numpy(X).to(dev()), [torch.zeros(n, F, device=dev()) for _ in range(12)]
        epp.epp_backward_aggregate(*work[F][:2], work[F][2][0])
        first[F] = work[F][2][0].clone()
        assert_close(first[F].cpu().numpy(), oracle.path_aggregate(n, paths_o[l], X), f"F={F}")
    streams = [torch.cuda.Stream() for _ in range(2)]
    for pair in zip(WIDTHS, WIDTHS[1:] + WIDTHS[:1]):
        for F in pair:
            for out in work[F][2]:
                out.zero_()
        torch.cuda.synchronize()
        for i in range(12):
            for F, s in zip(pair, streams):
                with torch.cuda.stream(s):
                    epp.epp_backward_aggregate(*work[F][:2], work[F][2][i])
        torch.cuda.synchronize()
        for F in pair:
            for i, out in enumerate(work[F][2]):
                assert torch.equal(out, first[F]), f"{pair}: F={F}, launch {i}"
    # a width that gives its count back and takes another way, and one that gets it
    p = work[16][0]
    p.set_group_size(16, 64)
    p.set_group_size(16, 0)
    for F in WIDTHS:
        epp.epp_backward_aggregate(*work[F][:2], work[F][2][0])
        assert torch.equal(work[F][2][0], first[F]), F
