"""Which kernel a launch runs on, around the limits of the row kernel's rule, and its results there against the group
kernel's: 16 M, 64 M and 100 M floats of gathered rows at whole and at broken lines."""
import numpy as np
import pytest
import torch

import paper_2204_02662_amd as epp
from _util import dev

pytestmark = pytest.mark.gpu

N, ROW = 60_000, 40


def _regular_graph():
    """ROW entries in every row but a few: one empty, some long ones."""
    rng = np.random.default_rng(5)
    lens = np.full(N, ROW)
    lens[[7, 1_000, 59_999]] = [0, 9_000, 3_000]
    rowptr = np.zeros(N + 1, np.int32)
    rowptr[1:] = np.cumsum(lens)
    col = np.concatenate([np.sort(rng.choice(N, size=k, replace=False)) if k > ROW else
                          (rng.integers(N) + np.sort(rng.choice(N // ROW, size=k, replace=False)) * ROW) % N for k in lens])
    order = np.lexsort((col, np.repeat(np.arange(N), lens)))
    return rowptr, col[order].astype(np.int32), (rng.standard_normal(col.size) / 6).astype(np.float32)


@pytest.mark.parametrize("F,rows", [(15, True), (16, True), (17, True), (24, True), (32, False), (41, True), (42, False), (47, False),
                                    (64, False)])
def test_rule_and_results(F, rows, monkeypatch):
    rowptr, col, val = (torch.from_numpy(a).to(dev()) for a in _regular_graph())
    assert 2.4e6 < col.numel() < 2.42e6  # (41 floats: 98.8 M, 42: 101.3 M; 32: 77 M)
    X = torch.randn(N, F, generator=torch.Generator(device="cuda").manual_seed(F), device="cuda")
    got = {}
    for mode in ("", "0"):
        monkeypatch.delenv("EPP_TUNE_ROWS", raising=False)
        if mode:
            monkeypatch.setenv("EPP_TUNE_ROWS", mode)
        train = torch.arange(0, N, 1, dtype=torch.int32, device="cuda")
        p = epp.epp_prepare(N, rowptr, col, val, train, 1).path(0)
        p.prepare_width(F)
        out = torch.full((N, F), 7.0, device="cuda")
        epp.epp_backward_aggregate(p, X, out)
        got[mode] = out
        assert (p.info().n_split_rows == 0) == (rows and not mode)  # (only the group table cuts the long rows)
    csr = torch.sparse_csr_tensor(rowptr, col, val.double(), (N, N))
    want, most = csr @ X.double(), torch.sparse_csr_tensor(rowptr, col, val.double().abs(), (N, N)) @ X.double().abs()
    want[7] = got["0"][7].double()  # (a row without entries)
    # a sum passes at most 32 additions in one lane, six between lanes, 36 of a long row's chunks: each rounds by 2^-24
    for mode, out in got.items():
        assert bool(((out.double() - want).abs() <= 128 * 2.0 ** -24 * most).all()), (F, mode)
    assert torch.equal(got[""][7], got["0"][7])


@pytest.mark.parametrize("n,row,F,rows", [
    (280_000, 30, 13, True), (280_000, 30, 14, False), (310_000, 40, 10, True), (310_000, 40, 13, False), (310_000, 40, 16, False),
    (290_000, 40, 16, True), (510_000, 40, 7, True), (510_000, 40, 10, False), (760_000, 40, 8, True), (760_000, 40, 7, False),
    (1_150_000, 3, 24, True), (1_200_000, 3, 24, False), (300_000, 6, 32, True), (320_000, 6, 32, False),
    (100_000, 7, 64, True), (110_000, 7, 64, False), (20_000, 22, 36, True), (20_000, 24, 36, False), (20_000, 60, 37, True)])
def test_limits(n, row, F, rows):
    """Either side of every limit, of entries, of gathered floats and of source floats: `row` equally spaced columns in every row."""
    r = torch.arange(n, device="cuda")[:, None]
    col = ((r * 7_919 + torch.arange(row, device="cuda") * (n // row)) % n).sort(1).values.int().reshape(-1)
    rowptr = torch.arange(0, n * row + 1, row, dtype=torch.int32, device="cuda")
    gen = torch.Generator(device="cuda").manual_seed(F)
    val = torch.randn(n * row, generator=gen, device="cuda")
    p = epp.epp_prepare(n, rowptr, col, val, torch.arange(n, dtype=torch.int32, device="cuda"), 1).path(0)
    p.prepare_width(F)
    assert (p.info().n_split_rows == 0) == rows
    X, Y = torch.randn(n, F, generator=gen, device="cuda"), torch.empty(n, F, device="cuda")
    epp.epp_backward_aggregate(p, X, Y)
    want = torch.sparse_csr_tensor(rowptr, col, val.double(), (n, n)) @ X.double()
    most = torch.sparse_csr_tensor(rowptr, col, val.double().abs(), (n, n)) @ X.double().abs()
    assert bool(((Y.double() - want).abs() <= (row + 2) * 2.0 ** -24 * most).all())


@pytest.mark.parametrize("switch,value", [("GS", 24), ("PACK", 0), ("PACK", 2), ("HOT_MB", 1)])
def test_switches_of_the_group_table_ask_for_it(switch, value, monkeypatch):
    rowptr, col, val = (torch.from_numpy(a).to(dev()) for a in _regular_graph())
    train = torch.arange(0, N, 1, dtype=torch.int32, device="cuda")
    p = epp.epp_prepare(N, rowptr, col, val, train, 1).path(0)
    monkeypatch.setenv(f"EPP_TUNE_{switch}", str(value))
    p.prepare_width(24)
    assert p.info().n_split_rows > 0 and (p.info().group_size == 24 or switch != "GS")
