"""Preparing a width while the caller's allocator refuses one block, whichever it is: the call either reports it, and
works when it is made again, or does without what the block was for.  Nothing is lost either way."""
import pytest

import graphgen
import oracle
import paper_2204_02662_amd as epp
from _util import assert_close, gpu_prepare, run_partial

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("F,env", [(47, {"EPP_TUNE_ROWS": "0", "EPP_TUNE_PACK": "2", "EPP_TUNE_PART": "2", "EPP_TUNE_HOT_MB": "1"}),
                                   (47, {"EPP_TUNE_ROWS": "0", "EPP_TUNE_PACK": "2", "EPP_TUNE_PART": "0"}),
                                   (64, {"EPP_TUNE_ROWS": "2"})])
def test_every_refused_block(F, env, monkeypatch):
    for k, v in {"EPP_TUNE_PART_KB": "16", "EPP_TUNE_PART_MINLEN": "8", "EPP_TUNE_SMALL_PREPARE": "0", **env}.items():
        monkeypatch.setenv(k, v)
    count, refused = [0], [-1]

    def alloc(nbytes, ctx):
        count[0] += 1
        return None if count[0] == refused[0] else epp._torch_alloc(nbytes, ctx)

    monkeypatch.setattr(epp, "_TORCH_ALLOC", epp._Alloc(epp._ALLOC_FN(alloc), epp._TORCH_ALLOC.free, None))
    g = graphgen.random_graph("rmat", 9_001, seed=601, raw_draws=120_000)
    train = graphgen.training_set(g.n, 3_000, 602)
    sets_o, paths_o = oracle.prepare(g.n, g.rowptr, g.col, g.val, train, 1)
    X = graphgen.normal_rows(g.n, F, sets_o[0], 603)
    want = oracle.path_aggregate(g.n, paths_o[0], X)
    live = epp.alloc_stats["live"]
    blocks, failed, k = None, 0, 0
    while blocks is None or k <= blocks:
        refused[0] = -1
        paths = gpu_prepare(g, train, 1)
        p = paths.path(0)
        count[0], refused[0] = 0, k
        try:
            p.prepare_width(F)
        except epp.EppError as e:
            assert e.code == epp.EPP_ERR_ALLOC
            failed += 1
            p.prepare_width(F)
        if blocks is None:
            blocks = count[0]
        refused[0] = -1
        assert_close(run_partial(p, X), want, f"block {k} of {blocks} refused")
        del p, paths
        assert epp.alloc_stats["live"] == live, f"block {k} of {blocks} refused"
        k += 1
    # the copy of the source rows and the partitioned layout are options; a plan of cut rows is not
    assert failed < blocks if env["EPP_TUNE_ROWS"] == "0" else failed == blocks
