"""The allocator that the library gets from the binding: what cannot be had is NULL and no exception, its counts, several threads."""
import threading

import pytest
import torch

import graphgen
import paper_2204_02662_amd as epp
from _util import gpu_prepare

pytestmark = pytest.mark.gpu


def test_refusal_and_counts():
    torch.zeros(1, device="cuda")
    before, held = dict(epp.alloc_stats), torch.cuda.memory_allocated()
    assert epp._torch_alloc(1 << 55) is None
    assert dict(epp.alloc_stats) == before
    p = epp._torch_alloc(1_000_000)
    assert p and p % 256 == 0 and torch.cuda.memory_allocated() >= held + 1_000_000
    now = dict(epp.alloc_stats)
    assert (now["allocs"], now["bytes"], now["live"]) == (before["allocs"] + 1, before["bytes"] + 1_000_000, before["live"] + 1)
    epp._torch_free(p)
    assert torch.cuda.memory_allocated() == held and epp.alloc_stats["live"] == before["live"]


def test_blocks_belong_to_the_callers_stream_in_every_thread():
    g = graphgen.random_graph("rmat", 9_001, seed=601, raw_draws=120_000)
    train = graphgen.training_set(g.n, 3_000, 602)
    want = [t.clone() for t in gpu_prepare(g, train, 2).path(0).export()]
    torch.cuda.synchronize()
    live, failed = epp.alloc_stats["live"], []

    def work():
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                for _ in range(8):
                    got = gpu_prepare(g, train, 2).path(0).export()
                    torch.cuda.current_stream().synchronize()
                    assert all(torch.equal(a, b) for a, b in zip(got, want))
        except BaseException as e:  # (an assertion in a thread is not seen otherwise)
            failed.append(e)

    threads = [threading.Thread(target=work) for _ in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not failed and epp.alloc_stats["live"] == live
