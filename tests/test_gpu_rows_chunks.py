"""Rows that the row kernel cuts into chunks: the last workgroup of such a row adds what the others have left, at the numbers of chunks
where its lanes take another share, launch after launch on other inputs, and replayed from a graph."""
import numpy as np
import pytest
import torch

import graphgen
import oracle
import paper_2204_02662_amd as epp
from _util import assert_close, dev

pytestmark = pytest.mark.gpu


def _lanes(F):
    lanes = 1
    while 4 * lanes < F and lanes < 64:
        lanes *= 2
    return lanes


@pytest.mark.parametrize("F", [3, 8, 16, 41, 64, 128, 259])
def test_rows_of_every_number_of_chunks(F, monkeypatch):
    monkeypatch.setenv("EPP_TUNE_ROWS", "2")
    lanes = _lanes(F)
    chunk, slots = 8192 // lanes, 256 // lanes
    counts = [2, 3, slots - 1, slots, slots + 1, 4 * slots, 4 * slots + 1]
    counts = [c for c in dict.fromkeys(counts) if 2 <= c <= 400_000 // chunk]
    lengths = [c * chunk - 3 for c in counts] + [chunk]
    n = max(lengths) + 8
    rng = np.random.default_rng(5)
    lens = np.ones(n, np.int64)
    lens[rng.permutation(n)[:len(lengths)]] = lengths
    rowptr = np.zeros(n + 1, np.int32)
    rowptr[1:] = np.cumsum(lens)
    col = np.concatenate([np.sort(rng.choice(n, size=k, replace=False)) for k in lens]).astype(np.int32)
    val = (rng.standard_normal(col.size) / np.sqrt(np.repeat(lens, lens))).astype(np.float32)
    train = np.arange(n, dtype=np.int32)
    sets_o, paths_o = oracle.prepare(n, rowptr, col, val, train, 1)
    d = dev()
    paths = epp.epp_prepare(n, *(torch.from_numpy(a).to(d) for a in (rowptr, col, val, train)), 1)
    p = paths.path(0)
    p.prepare_width(F)
    X = [graphgen.normal_rows(n, F, sets_o[0], 12 + i) for i in range(3)]
    want = [oracle.path_aggregate(n, paths_o[0], x) for x in X]
    X = [torch.from_numpy(x).to(d) for x in X]
    first = []
    for i in range(3):
        out = torch.full((n, F), float("nan"), device=d)
        epp.epp_backward_aggregate(p, X[i], out)
        assert_close(out.cpu().numpy(), want[i], f"F={F} input {i}")
        first.append(out)
    # one launch behind the other: no sum of the launch before is taken for one of this
    outs = [torch.full((n, F), float("nan"), device=d) for _ in range(24)]
    for i, out in enumerate(outs):
        epp.epp_backward_aggregate(p, X[i % 3], out)
    for i, out in enumerate(outs):
        assert torch.equal(out, first[i % 3]), i
    # from a graph, with other launches between the replays
    x, out = X[0].clone(), torch.empty(n, F, device=d)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        epp.epp_backward_aggregate(p, x, out)
    for i in (1, 2, 0, 1):
        x.copy_(X[i])
        out.fill_(float("nan"))
        graph.replay()
        epp.epp_backward_aggregate(p, X[0], outs[0])
        torch.cuda.synchronize()
        assert torch.equal(out, first[i]) and torch.equal(outs[0], first[0]), i
