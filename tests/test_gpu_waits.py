"""Calls that synchronise their stream: the runtime knows it, too, as soon as they are back."""
import pytest
import torch

import paper_2204_02662_amd as epp
from _util import dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("own", [False, True])
@pytest.mark.parametrize("n,per_row,F", [(9_000, 4, 16), (66_000, 8, 41), (66_000, 150, 64)])
def test_the_stream_is_idle(n, per_row, F, own, monkeypatch):
    monkeypatch.setenv("EPP_TUNE_SMALL_PREPARE", "0")  # (the one-launch preparation waits for its kernel, not for the stream)
    gen = torch.Generator(dev()).manual_seed(n + F)
    nnz = n * per_row
    col = torch.randint(0, n, (nnz,), device=dev(), generator=gen).int()
    rowptr = torch.arange(0, nnz + 1, per_row, dtype=torch.int32, device=dev())
    rowptr[1:n // 2] = rowptr[n // 2].clone()  # (one very long row, many without entries)
    val = torch.ones(nnz, device=dev())
    train = torch.arange(0, n, 9, dtype=torch.int32, device=dev())
    torch.cuda.synchronize()
    with torch.cuda.stream(torch.cuda.Stream() if own else torch.cuda.current_stream()):
        def idle(what, x):
            assert torch.cuda.current_stream().query(), what
            return x
        for _ in range(3):
            paths = idle("prepare", epp.epp_prepare(n, rowptr, col, val, train, 2))
            full = idle("prepare_full", epp.epp_prepare_full(n, rowptr, col, val))
            saved = [idle("export", paths.path(l).export()) for l in range(2)]
            again = idle("import", epp.epp_paths_import(n, train, saved))
            for p in (paths.path(0), full, again.path(1), again.path(0)):
                idle("prepare_width", p.prepare_width(F))
            idle("active_set", paths.active_set(1))
