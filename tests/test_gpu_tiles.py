"""Launches on tiles of rows whose sums stay in LDS (csrc/epp_tiles.hip), forced onto small graphs: widths at the ends of
slices and lines, cut rows, batches that hold a row many times, tiles that are sorted in several rounds, paths that run on
the next outer path's tiles.  512 tiles at a time instead of 2,048, so that a graph of this size fills them."""
import numpy as np
import pytest
import torch

import graphgen
import oracle
import paper_2204_02662_amd as epp
from _util import assert_close, assert_paths_bit_exact, dev, gpu_prepare, gpu_prepare_full, run_full, run_ifelse, run_partial

pytestmark = pytest.mark.gpu

_ALLOCATORS = []  # (handles that a failed test leaves behind give their memory back through them)


def _force(monkeypatch, lanes, split=512, **more):
    for k, v in {"ROWS": "0", "TILES": "2", "TILE_LANES": lanes, "TILE_SPLIT": split, "TILES_AT_ONCE": 512,
                 "SMALL_PREPARE": "0", **more}.items():
        monkeypatch.setenv("EPP_TUNE_" + k, str(v))


@pytest.mark.parametrize("lanes", [4, 8, 16])
@pytest.mark.parametrize("split", [16, 512])
def test_every_width_shared_and_own_entries(lanes, split, monkeypatch):
    """Two generations of tiles; the inner path runs on the outer one's, at any overlap."""
    g = graphgen.random_graph("rmat", 90_001, seed=71, raw_draws=700_000)
    train = graphgen.training_set(g.n, 9_000, 72)
    sets_o, paths_o = oracle.prepare(g.n, g.rowptr, g.col, g.val, train, 2)
    for share in ("1", "0"):
        _force(monkeypatch, lanes, split, SHARE_PCT=share)
        paths = gpu_prepare(g, train, 2)
        assert [paths.path(l).info().shares_entries for l in (0, 1)] == [0, int(share)]
        for F in (5, 8, 15, 16, 17, 31, 32, 33, 47, 64, 65, 100, 128, 259):
            for l in (1, 0):
                src, rows = sets_o[1 - l].astype(bool), sets_o[2 - l].astype(bool)
                X = graphgen.normal_rows(g.n, F, sets_o[1 - l], 73 + l)
                want = oracle.path_aggregate(g.n, paths_o[l], X)
                X[~src] = np.nan  # never read
                p = paths.path(l)
                got = run_partial(p, X, poison=9.0)
                what = f"lanes={lanes} split={split} share={share} F={F} l={l}"
                assert np.all(got[~rows] == 9.0), what
                assert_close(got[rows], want[rows], what)
                assert np.array_equal(got[rows], run_partial(p, X, poison=1.0)[rows]), what
                i = p.info()
                longest = np.diff(paths_o[0 if share == "1" else l].rowptr).max()
                assert (i.part_rows > 0) == (longest > split) and i.part_partial_rows >= 2 * i.part_rows, what
        assert_paths_bit_exact(paths, sets_o, paths_o, 2)


@pytest.mark.parametrize("lanes", [4, 8, 16])
@pytest.mark.parametrize("n,draws", [(700, 60_000), (2_500, 900_000), (90_000, 5_000_000)])
def test_dense_rows_and_large_tiles(lanes, n, draws, monkeypatch):
    """Rows that have many of a batch's entries (all levels of care), and tiles of several rounds; a second handle gives the
    same bits; the if-else baseline of the same handle still runs on its group table."""
    _force(monkeypatch, lanes)
    g = graphgen.random_graph("rmat", n, seed=81, raw_draws=draws)
    F = 20
    X = graphgen.normal_rows(g.n, F, None, 82)
    want = oracle.full_aggregate(g.n, g.rowptr, g.col, g.val, X)
    full = gpu_prepare_full(g)
    got = run_full(full, X)
    assert_close(got, want, f"lanes={lanes} n={n}")
    assert np.array_equal(got, run_full(gpu_prepare_full(g), X))
    paths = gpu_prepare(g, np.arange(g.n, dtype=np.int32), 1)
    assert_close(run_ifelse(full, paths, 0, X), want, "if-else")


@pytest.mark.parametrize("lanes", [4, 8, 16])
def test_columns_in_any_order(lanes, monkeypatch):
    """A tile of one round needs no order of the columns; one of several rounds does, and the path then keeps its group table."""
    _force(monkeypatch, lanes)
    rng = np.random.default_rng(91)
    for n, draws, tiles in ((20_000, 200_000, True), (90_000, 5_000_000, False)):
        g = graphgen.random_graph("rmat", n, seed=92, raw_draws=draws)
        row = np.repeat(np.arange(g.n), np.diff(g.rowptr))
        order = np.lexsort((rng.random(g.nnz), row))
        col, val = g.col[order].copy(), g.val[order].copy()
        X = graphgen.normal_rows(g.n, 33, None, 93)
        want = oracle.full_aggregate(g.n, g.rowptr, col, val, X)
        full = epp.epp_prepare_full(g.n, *(torch.from_numpy(x).to(dev()) for x in (g.rowptr, col, val)))
        assert_close(run_full(full, X), want, f"lanes={lanes} n={n}")
        assert (full.info().part_rows > 0) == (tiles and np.diff(g.rowptr).max() > 512)


@pytest.mark.parametrize("lanes", [4, 8, 16])
def test_entries_that_do_not_fit_are_laid_out_once(lanes, monkeypatch):
    """Rows whose columns do not ascend, in tiles of several rounds: the first width finds out, the next one of the same lanes takes
    no memory for tiles."""
    _force(monkeypatch, lanes, PACK=0, PART=0)
    g = graphgen.random_graph("rmat", 90_000, seed=92, raw_draws=5_000_000)
    order = np.lexsort((np.random.default_rng(91).random(g.nnz), np.repeat(np.arange(g.n), np.diff(g.rowptr))))
    col, val = g.col[order].copy(), g.val[order].copy()
    paths = epp.epp_prepare(g.n, *(torch.from_numpy(x).to(dev()) for x in (g.rowptr, col, val)),
                            torch.arange(g.n, dtype=torch.int32, device=dev()), 1)
    taken = []
    for F in (33, 47):
        before = epp.alloc_stats["bytes"]
        paths.path(0).prepare_width(F)
        taken.append(epp.alloc_stats["bytes"] - before)
        X = graphgen.normal_rows(g.n, F, None, 93)
        assert_close(run_partial(paths.path(0), X)[np.diff(g.rowptr) > 0],
                     oracle.full_aggregate(g.n, g.rowptr, col, val, X)[np.diff(g.rowptr) > 0], f"lanes={lanes} F={F}")
    assert taken[0] > 8 * g.nnz > taken[1], taken


@pytest.mark.parametrize("lanes", [4, 8, 16])
@pytest.mark.parametrize("F", [16, 47])
def test_infinities_stay_where_they_belong(lanes, F, monkeypatch):
    _force(monkeypatch, lanes)
    g = graphgen.random_graph("chung_lu", 40_000, seed=95, target_edges=150_000)
    X = graphgen.normal_rows(g.n, F, None, 96)
    X[::977] = np.inf
    X[5::1201] = -np.inf
    X[7::3001, 0] = np.nan
    with np.errstate(invalid="ignore"):
        want = oracle.full_aggregate(g.n, g.rowptr, g.col, g.val, X)
    got = run_full(gpu_prepare_full(g), X)
    ok = np.isfinite(want)
    assert np.array_equal(np.isnan(got), np.isnan(want)) and np.array_equal(got[~ok & ~np.isnan(want)], want[~ok & ~np.isnan(want)])
    assert_close(got[ok], want[ok], f"lanes={lanes} F={F}")


@pytest.mark.parametrize("F", [47, 64])
def test_captured_launches(F, monkeypatch):
    _force(monkeypatch, 8, 32)
    g = graphgen.random_graph("rmat", 60_000, seed=97, raw_draws=500_000)
    full = gpu_prepare_full(g)
    full.prepare_width(F)
    x = torch.zeros(g.n, F, device=dev())
    y, z = torch.empty_like(x), torch.empty_like(x)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        epp.epp_full_aggregate(full, x, y)
    for rep in range(3):
        x.normal_()
        graph.replay()
        torch.cuda.synchronize()
        epp.epp_full_aggregate(full, x, z)
        assert torch.equal(y, z), f"replay {rep}"
    assert_close(y.cpu().numpy(), oracle.full_aggregate(g.n, g.rowptr, g.col, g.val, x.cpu().numpy()), f"F={F}")


@pytest.mark.parametrize("F", [47, 64])
def test_every_refused_block(F, monkeypatch):
    """Tiles are an option: without memory for them, for the parts' sums or for the copy, the group table serves."""
    _force(monkeypatch, 8, 32)
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
    blocks, k = None, 0
    while blocks is None or k <= blocks:
        refused[0] = -1
        paths = gpu_prepare(g, train, 1)
        p = paths.path(0)
        count[0], refused[0] = 0, k
        p.prepare_width(F)
        blocks = count[0] if blocks is None else blocks
        refused[0] = -1
        assert (p.info().part_rows > 0) == (k == 0), f"block {k} of {blocks} refused"
        assert_close(run_partial(p, X), want, f"block {k} of {blocks} refused")
        p.set_group_size(F, 24)
        assert_close(run_partial(p, X), want, "group table asked for")
        p.set_group_size(F, 0)
        assert p.info().part_rows > 0
        assert_close(run_partial(p, X), want, "tiles again")
        del p, paths
        assert epp.alloc_stats["live"] == live, f"block {k} of {blocks} refused"
        k += 1


def _ordered_graph(order):
    """23 M entries among 400,000 vertices: hubs and their neighbours anywhere ("random") or in front ("degree"), or all neighbours
    within 300 ids ("band")."""
    n, gen = 400_000, torch.Generator(device="cuda").manual_seed(7)
    u, v = ((torch.rand(13_000_000, generator=gen, device="cuda", dtype=torch.float64) ** 4 * n).long() for _ in range(2))
    if order == "band":
        v = (u + torch.randint(1, 300, u.shape, generator=gen, device="cuda")) % n
    elif order == "random":
        ids = torch.randperm(n, generator=gen, device="cuda")
        u, v = ids[u], ids[v]
    keys = torch.unique(torch.cat((u * n + v, v * n + u)))
    row, col = keys // n, (keys % n).int()
    rowptr = torch.zeros(n + 1, dtype=torch.int32, device="cuda")
    rowptr[1:] = torch.cumsum(torch.bincount(row, minlength=n), 0)
    val = torch.randn(col.shape, generator=gen, device="cuda")
    path = epp.epp_prepare(n, rowptr, col, val, torch.arange(n, dtype=torch.int32, device="cuda"), 1).path(0)
    return n, rowptr, col, val, path


@pytest.mark.parametrize("order,tiles", [("random", True), ("band", False), ("degree", False)])
def test_ids_in_an_order_stay_on_the_group_table(order, tiles):
    """By the library's own rule, paths run on tiles where neighbours lie anywhere, but not where rows have theirs close together and
    the entries of a batch would wait for each other."""
    F, gen = 64, torch.Generator(device="cuda").manual_seed(8)
    n, rowptr, col, val, path = _ordered_graph(order)
    X, Y = torch.randn(n, F, generator=gen, device="cuda"), torch.zeros(n, F, device="cuda")
    path.prepare_width(F)
    epp.epp_backward_aggregate(path, X, Y)
    assert (path.info().n_split_rows == 0) == tiles  # (only the group table has groups that cut rows)
    want = torch.sparse_csr_tensor(rowptr, col, val.double(), (n, n)) @ X.double()
    most = torch.sparse_csr_tensor(rowptr, col, val.double().abs(), (n, n)) @ X.double().abs()
    # chains of 512 additions, and at most n / 512 of their sums: each addition rounds by 2^-24
    assert bool(((Y.double() - want).abs() <= (512 + n / 512) * 2.0 ** -24 * most).all())


@pytest.mark.parametrize("switch,value", [("GS", 96), ("PACK", 0), ("PACK", 2), ("PART", 2), ("HOT_MB", 1), ("LOG2_SLICES", 1)])
def test_switches_of_the_group_table_ask_for_it(switch, value, monkeypatch):
    monkeypatch.setenv(f"EPP_TUNE_{switch}", str(value))
    path = _ordered_graph("random")[-1]
    path.prepare_width(64)
    i = path.info()
    assert i.n_split_rows > 0
    assert i.group_size == 96 or switch != "GS"
    assert i.part_hot_entries > 0 or switch != "PART"


@pytest.mark.parametrize("F", [47, 64])
@pytest.mark.parametrize("all_active", [False, True])
def test_memory_for_the_group_table_is_enough(F, all_active, monkeypatch):
    """Whatever lies between what the group table needs and what the tiles take: the width is prepared, and nothing is left over."""
    sizes, live, peak, budget = {}, [0], [0], [1 << 60]

    def alloc(nbytes, ctx):
        p = epp._torch_alloc(nbytes, ctx) if live[0] + nbytes <= budget[0] else None
        if p:
            sizes[p] = nbytes
            live[0] += nbytes
            peak[0] = max(peak[0], live[0])
        return p

    def free(ptr, ctx):
        live[0] -= sizes.pop(ptr)
        epp._torch_free(ptr, ctx)

    _ALLOCATORS.append(epp._Alloc(epp._ALLOC_FN(alloc), epp._FREE_FN(free), None))
    monkeypatch.setattr(epp, "_TORCH_ALLOC", _ALLOCATORS[-1])
    g = graphgen.random_graph("rmat", 40_001, seed=611, raw_draws=900_000)
    train = np.arange(g.n, dtype=np.int32)
    X = graphgen.normal_rows(g.n, F, None, 612)
    want = oracle.full_aggregate(g.n, g.rowptr, g.col, g.val, X)
    some = np.diff(g.rowptr) > 0

    def prepared(tiles, limit):
        """Bytes that preparing the width took at most, and whether it has tiles."""
        _force(monkeypatch, 8, 32, TILES=tiles, PACK=0, PART=0)
        handle = gpu_prepare_full(g) if all_active else gpu_prepare(g, train, 1)
        p = handle if all_active else handle.path(0)
        base = peak[0] = live[0]
        budget[0] = base + limit
        p.prepare_width(F)
        budget[0] = 1 << 60
        most, cut = peak[0] - base, p.info().part_rows
        got = run_full(p, X) if all_active else run_partial(p, X)
        assert_close(got[some], want[some], f"limit {limit}")
        if all_active and limit < 1 << 50:
            assert_close(run_ifelse(p, gpu_prepare(g, train, 1), 0, X)[some], want[some], f"if-else, limit {limit}")
        del p, handle
        assert live[0] == 0
        return most, cut > 0

    groups, with_tiles = prepared(0, 1 << 59)[0], prepared(2, 1 << 59)[0]
    assert groups < with_tiles
    limits = np.linspace(groups, with_tiles, 25).astype(np.int64).tolist()
    assert [prepared(2, limit)[1] for limit in (limits[0], limits[-1])] == [False, True]
    for limit in limits[1:-1]:
        prepared(2, limit)


def test_report_of_a_path_that_was_prepared_through_its_inner_one(monkeypatch):
    _force(monkeypatch, 8, SHARE_PCT=1)
    g = graphgen.random_graph("rmat", 20_000, seed=621, raw_draws=200_000)
    paths = gpu_prepare(g, graphgen.training_set(g.n, 4_000, 622), 2)
    assert paths.path(1).info().shares_entries
    paths.path(1).prepare_width(20)
    assert [paths.path(l).info().sched_F for l in (0, 1)] == [20, 20]
    assert paths.path(0).info().n_split_rows == 0 and paths.path(0).info().group_size == paths.path(0).select_group_size(20)


@pytest.mark.parametrize("lanes", [4, 8, 16])
def test_sums_of_rows_with_neighbouring_sources(lanes, monkeypatch):
    """600 rows of 500 consecutive columns among rows of 8 columns anywhere: all of a row's entries meet in one part of the sweep,
    so that its sum is one chain of additions, the longest there can be."""
    _force(monkeypatch, lanes)
    n, F, rng = 30_000, 24, np.random.default_rng(631)
    cols = [np.sort(rng.choice(n, 8, replace=False)) for _ in range(n)]
    for r in rng.choice(n, 600, replace=False):
        cols[r] = rng.integers(n - 500) + np.arange(500)
    rowptr = np.zeros(n + 1, np.int32)
    rowptr[1:] = np.cumsum([c.size for c in cols])
    col = np.concatenate(cols).astype(np.int32)
    val = rng.random(col.size).astype(np.float32)  # all positive, like the inputs: sums grow, the worst case for a chain
    X = rng.random((n, F)).astype(np.float32)
    full = epp.epp_prepare_full(n, *(torch.from_numpy(a).to(dev()) for a in (rowptr, col, val)))
    got = run_full(full, X).astype(np.float64)
    want = np.add.reduceat(val[:, None].astype(np.float64) * X[col], rowptr[:-1])
    # each of the at most 512 + 16 additions (fused with its product) rounds by 2^-24 of what is there by then, at most the sum
    assert (np.abs(got - want) <= 528 * 2.0 ** -24 * want).all()
    # and the errors of a chain hardly ever add up: 2-norms, 2^-24 times sqrt(500 / 3) on average
    assert np.linalg.norm(got - want) <= 4 * np.sqrt(500 / 3) * 2.0 ** -24 * np.linalg.norm(want)


@pytest.mark.parametrize("n,tiles", [(1 << 23, True), (1 + (1 << 23), False)])
def test_ids_of_more_than_23_bits_stay_on_the_group_table(n, tiles, monkeypatch):
    """60,000 rows among the first and last ids, columns anywhere, the last id among them."""
    _force(monkeypatch, 8)
    F, gen = 20, torch.Generator(device="cuda").manual_seed(641)
    rows = torch.cat((torch.arange(30_000, device="cuda"), torch.arange(n - 30_000, n, device="cuda")))
    col = torch.randint(n, (60_000, 9), generator=gen, device="cuda")
    col[:, 8] = n - 1
    row, col = (x.reshape(-1) for x in torch.broadcast_tensors(rows[:, None], col))
    keys = torch.unique(row * n + col)
    row, col = keys // n, (keys % n).int()
    rowptr = torch.zeros(n + 1, dtype=torch.int32, device="cuda")
    rowptr[1:] = torch.cumsum(torch.bincount(row, minlength=n), 0)
    val = torch.rand(col.shape, generator=gen, device="cuda")
    path = epp.epp_prepare(n, rowptr, col, val, torch.arange(n, dtype=torch.int32, device="cuda"), 1).path(0)
    X, Y = torch.rand(n, F, generator=gen, device="cuda"), torch.full((n, F), 7.0, device="cuda")
    path.prepare_width(F)
    assert (path.info().n_split_rows == 0) == tiles
    epp.epp_backward_aggregate(path, X, Y)
    want = torch.zeros(n, F, dtype=torch.float64, device="cuda").index_add_(0, row, val.double()[:, None] * X[col.long()].double())
    assert bool((Y[30_000:n - 30_000] == 7.0).all())
    # nine positive terms: eleven additions at most, each rounds by 2^-24 of what is there by then
    assert bool(((Y.double() - want).abs() <= 11 * 2.0 ** -24 * want)[rows].all())
