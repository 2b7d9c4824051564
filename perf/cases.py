"""Workloads of the library, as a training program calls it.

A case is one pass over one synthetic graph: symmetric, with self-loops, vertex ids in random order, weights
1/sqrt(d_v d_u), generated on the GPU.  The seed of `prepare` numbers the vertices and draws all gradients, forward
results and weights; who is connected to whom and who trains is the case's own, so that array sizes do not depend on
the seed.  What a pass does (`op`):

  epoch        backward aggregation of every layer over prepared paths (the inner loop of training);
               with `captured` the same launches replayed from a HIP graph, as launch-bound loops do
  full         all-active aggregation of every layer (forward propagation, or training on all vertices)
  backward     the whole backward loop: weight gradient, input gradient and aggregation of every layer, chained;
               with `static` the weight gradient uses the library's own scratch instead of a workspace
  combine      weight and input gradient of every layer over the active rows
  first_epoch  paths prepared on the fly: path construction, width preparation, then one epoch
  preprocess   path construction and export of every path (prepare once, save, reuse)
  resume       import of saved paths, width preparation, then one epoch

`widths` lists the gradient width of layer 0, 1, ... L-1 (layer L-1 runs first and has the training set as its
sources); a layer's weight matrix is F_l x F_{l+1}, with F_L = F_{L-1}.
"""
import math

import torch

import paper_2204_02662_amd as epp

RMAT = (0.57, 0.19, 0.19)
GAMMA = 2.5  # exponent of the power-law degrees of the Chung-Lu model
LARGEST_GATHER = 6.8e10  # gathered floats of the largest listed pass (the stress graph's epoch)


def _case(name, op, model, n, edges, train, widths, **more):
    c = {"name": name, "op": op, "model": model, "n": n, "edges": edges, "train": train, "biased": False,
         "widths": " ".join(map(str, widths)), "captured": False, "static": False}
    c.update(more)
    return c


def listed():
    citation = ("chung_lu", 2_708, 5_278, 140, (16, 7))
    sparse = ("chung_lu", 19_717, 44_324, 60, (16, 3))
    social = ("rmat", 232_965, 57_300_000, 153_757, (16, 41))
    copurchase = ("chung_lu", 2_449_029, 61_900_000, 196_615, (64, 64, 47))
    stress = ("rmat", 1 << 23, 129_300_000, 83_886, (128, 128, 16))
    return [
        # a citation graph: every kernel is shorter than its launch
        _case("epoch citation", "epoch", *citation),
        # a few training vertices in a sparse graph, the epoch captured once and replayed
        _case("epoch sparse captured", "epoch", *sparse, captured=True),
        # the backward loop on the same graph, nothing allocated and no workspace
        _case("backward sparse", "backward", *sparse, static=True),
        # dense social graph, narrow rows of odd width, most vertices train
        _case("epoch social", "epoch", *social),
        # large sparse graph, 8 % train, rows of 188 and 256 bytes
        _case("epoch copurchase", "epoch", *copurchase),
        # the largest: extreme degree skew, 512-byte rows
        _case("epoch stress", "epoch", *stress, biased=True),
        # all-active aggregation of the same layers as "epoch copurchase"
        _case("full copurchase", "full", *copurchase),
        # whole backward loop of a two-layer model on a mid-size social network, 10 % train, 41 classes
        _case("backward community", "backward", "rmat", 1_134_890, 2_987_624, 113_489, (16, 41)),
        # dense products over the active rows only, up to 4.6 M rows of 128
        _case("combine stress", "combine", *stress, biased=True),
        # a short run on a small graph prepares its paths inside the first epoch
        _case("first epoch citation", "first_epoch", *citation),
        # paths of the co-purchase graph built and saved
        _case("preprocess copurchase", "preprocess", *copurchase),
        # saved paths of a mid-size blog network loaded for a new run
        _case("resume blog", "resume", "chung_lu", 88_784, 2_093_195, 8_878, (16, 39)),
    ]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _draw_width(rng):
    if rng.random() < 0.5:
        return rng.choice((16, 32, 64, 128))  # hidden layers
    return round(_log_uniform(rng, 2, 160))   # class counts and feature widths of any size


def draw(rng):
    while True:
        n = round(_log_uniform(rng, 500, 1 << 23))
        degree = _log_uniform(rng, 2, 250)  # undirected edges per vertex
        model = rng.choice(("chung_lu", "rmat"))
        edges = round(n * min(degree, n / 40))
        if edges > 129_300_000:
            continue
        layers = rng.choice((2, 2, 2, 3, 3, 4))
        op = rng.choice(("epoch", "epoch", "epoch", "backward", "backward", "full", "combine", "first_epoch",
                         "preprocess", "resume"))
        train = max(1, round(n * _log_uniform(rng, 0.003, 0.66)))
        hidden = _draw_width(rng)
        widths = [hidden] * (layers - 1) + [_draw_width(rng)]
        c = _case("", op, model, n, edges, train, widths, biased=rng.random() < 0.25,
                  captured=op == "epoch" and rng.random() < 0.25, static=op == "backward" and rng.random() < 0.5)
        del c["name"]
        if (2 * edges + n) * sum(widths) <= LARGEST_GATHER:
            return c


# ---------------------------------------------------------------------------------------------- inputs
def _pairs(case, m, gen):
    """m random vertex pairs of the model, as two int64 tensors; pairs with an id >= n are left out."""
    n = case["n"]
    if case["model"] == "chung_lu":  # P(i) ~ (i+1)^(-1/(GAMMA-1)): inverse of the distribution function
        power = (GAMMA - 1.0) / (GAMMA - 2.0)
        u, v = ((torch.rand(m, generator=gen, device="cuda", dtype=torch.float64).pow_(power).mul_(n)).long().clamp_(max=n - 1)
                for _ in range(2))
        return u, v
    a, b, c = RMAT
    u = torch.zeros(m, dtype=torch.int32, device="cuda")
    v = torch.zeros(m, dtype=torch.int32, device="cuda")
    for _ in range(max(1, (n - 1).bit_length())):
        x = torch.rand(m, generator=gen, device="cuda")
        low = x >= a + b
        right = ((x >= a) & ~low) | (x >= a + b + c)
        u.mul_(2).add_(low)
        v.mul_(2).add_(right)
    inside = (u < n) & (v < n)
    return u[inside].long(), v[inside].long()


def _graph(case, order, gen):
    """(rowptr, col, val, degree) of the normalised adjacency matrix with self-loops; vertex i gets the id order[i]."""
    n, target = case["n"], case["edges"]
    keys = torch.empty(0, dtype=torch.int64, device="cuda")
    for _ in range(24):  # duplicates are drawn again, until about `edges` distinct ones are there
        missing = target - keys.numel()
        if missing <= target // 100:
            break
        u, v = _pairs(case, missing + missing // 8 + 16, gen)
        new = (torch.minimum(u, v) * n + torch.maximum(u, v))[u != v]
        del u, v
        keys = torch.unique(torch.cat((keys, new)) if keys.numel() else new)
        del new
    u, v = order[keys // n], order[keys % n]
    loops = torch.arange(n, device="cuda", dtype=torch.int64)
    keys = torch.cat((u * n + v, v * n + u, loops * (n + 1)))
    del u, v
    keys = torch.sort(keys).values
    row, col = keys // n, (keys % n).int()
    del keys
    degree = torch.bincount(row, minlength=n)
    rowptr = torch.zeros(n + 1, dtype=torch.int32, device="cuda")
    rowptr[1:] = torch.cumsum(degree, 0)
    scale = degree.double().rsqrt()
    val = (scale[row] * scale[col.long()]).float()
    return rowptr, col, val, degree


def _train_ids(case, order, degree, gen):
    n, count = case["n"], case["train"]
    if not case["biased"]:
        return order[torch.randperm(n, generator=gen, device="cuda")[:count]].int()
    keys = torch.rand(n, generator=gen, device="cuda", dtype=torch.float64).log_().div_(degree[order])  # P(v) ~ degree
    return order[torch.topk(keys, count).indices].int()


def _widths(case):
    w = [int(x) for x in case["widths"].split()]
    return w, w + [w[-1]]


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    n, op = case["n"], case["op"]
    widths, wide = _widths(case)
    L = len(widths)
    structure = torch.Generator(device="cuda")
    structure.manual_seed(2204)
    order = torch.randperm(n, generator=gen, device="cuda")
    rowptr, col, val, degree = _graph(case, order, structure)
    train = _train_ids(case, order, degree, structure)
    del order, degree
    s = {"case": case, "widths": widths, "L": L}

    def normal(F, rows=None):
        """n x F of N(0,1); on the given rows only, zeros elsewhere, as an active set's gradients are."""
        if rows is None:
            return torch.randn(n, F, generator=gen, device="cuda")
        x = torch.zeros(n, F, device="cuda")
        x[rows] = torch.randn(rows.numel(), F, generator=gen, device="cuda")
        return x

    if op in ("preprocess", "first_epoch"):
        s["csr"] = (n, rowptr, col, val, train)
        if op == "preprocess":
            return s
    paths = epp.epp_prepare(n, rowptr, col, val, train, L)
    sets = [paths.active_set(k).long() for k in range(L)]
    if op in ("epoch", "full", "first_epoch", "resume"):
        # gradients of layer l live on the sources N^(L-l-1) of its path; the all-active operator takes any matrix
        s["in"] = [normal(widths[l], None if op == "full" else sets[L - l - 1]) for l in range(L)]
        s["out"] = [torch.zeros(n, widths[l], device="cuda") for l in range(L)]
    if op == "full":
        s["full"] = epp.epp_prepare_full(n, rowptr, col, val)
        for F in widths:
            s["full"].prepare_width(F)
        return s
    if op == "first_epoch":
        return s
    if op == "resume":
        s["saved"] = [paths.path(l).export() for l in range(L)]
        s["train"] = train
        return s
    s["paths"] = paths
    s["path"] = [paths.path(l) for l in range(L)]
    if op in ("epoch", "backward"):
        for l in range(L):
            s["path"][l].prepare_width(widths[l])
    if op in ("combine", "backward"):
        s["Y"] = [normal(wide[l]) for l in range(L)]  # forward aggregation results
        s["W"] = [torch.randn(wide[l], wide[l + 1], generator=gen, device="cuda") / math.sqrt(wide[l + 1]) for l in range(L)]
        s["gW"] = [torch.empty(wide[l], wide[l + 1], device="cuda") for l in range(L)]
        s["gY"] = [torch.zeros(n, wide[l], device="cuda") for l in range(L)]
        if op == "combine":
            s["gX"] = [normal(wide[l + 1], sets[L - l - 1]) for l in range(L)]
        else:  # gX[L] comes from the loss, gX[l] from the aggregation of layer l
            s["gX"] = [torch.zeros(n, wide[l], device="cuda") for l in range(L)] + [normal(wide[L], sets[0])]
        if not case["static"]:
            size = max(epp.epp_weight_gradient_workspace(paths, L - l - 1, wide[l], wide[l + 1]) for l in range(L))
            s["ws"] = torch.empty(size, dtype=torch.uint8, device="cuda")
    if case["captured"]:
        s["graph"] = torch.cuda.CUDAGraph()
        torch.cuda.synchronize()
        with torch.cuda.graph(s["graph"]):
            _epoch(s)
    return s


# ------------------------------------------------------------------------------------------------- passes
def _epoch(s):
    for l in range(s["L"] - 1, -1, -1):
        epp.epp_backward_aggregate(s["path"][l], s["in"][l], s["out"][l])


def _combine(s, l, gX):
    k = s["L"] - l - 1
    if s["case"]["static"]:
        epp.epp_weight_gradient_static(s["paths"], k, s["Y"][l], gX, s["gW"][l])
    else:
        epp.epp_weight_gradient(s["paths"], k, s["Y"][l], gX, s["gW"][l], s["ws"])
    epp.epp_input_gradient(s["paths"], k, gX, s["W"][l], s["gY"][l])


def run(s):
    op, L = s["case"]["op"], s["L"]
    if op == "epoch":
        if "graph" in s:
            s["graph"].replay()
        else:
            _epoch(s)
        return s["out"]
    if op == "full":
        for l in range(L - 1, -1, -1):
            epp.epp_full_aggregate(s["full"], s["in"][l], s["out"][l])
        return s["out"]
    if op == "backward":
        for l in range(L - 1, -1, -1):
            _combine(s, l, s["gX"][l + 1])
            epp.epp_backward_aggregate(s["path"][l], s["gY"][l], s["gX"][l])
        return {"gW": s["gW"], "gX": s["gX"][:L]}
    if op == "combine":
        for l in range(L - 1, -1, -1):
            _combine(s, l, s["gX"][l])
        return {"gW": s["gW"], "gY": s["gY"]}
    if op == "preprocess":
        paths = epp.epp_prepare(*s["csr"], L)
        return [paths.path(l).export() for l in range(L)]
    # a run that begins: the handle stays with the program, the one of the pass before is given back
    paths = epp.epp_prepare(*s["csr"], L) if op == "first_epoch" else epp.epp_paths_import(s["case"]["n"], s["train"], s["saved"])
    s["paths"], s["path"] = paths, [paths.path(l) for l in range(L)]
    for l in range(L):
        s["path"][l].prepare_width(s["widths"][l])
    _epoch(s)
    return s["out"]


# ------------------------------------------------------------------------------------------- work and tolerance
def _expected_sizes(case):
    """(entries of the graph, |N^k| for k = 0..L, entries of the path with sources N^k for k = 0..L-1): mean-field
    expectation over the degree classes of the model."""
    n, E = case["n"], case["edges"]
    if case["model"] == "rmat":
        bits = max(1, (n - 1).bit_length())
        one = RMAT[0] + RMAT[1]
        classes = [(n * math.comb(bits, z) / 2.0 ** bits, one ** (bits - z) * (1 - one) ** z) for z in range(bits + 1)]
    else:  # 96 slices of the vertices, equal in the logarithm of the rank
        edge = [math.exp(math.log(n + 1) * i / 96) for i in range(97)]
        classes = [(b - a, math.sqrt(a * b) ** (-1.0 / (GAMMA - 1))) for a, b in zip(edge, edge[1:])]
    total = sum(c * w for c, w in classes)
    classes = [(c, min(n - 1.0, 2.0 * E * w / total) + 1.0) for c, w in classes]
    nnz = sum(c * d for c, d in classes)
    p = [min(1.0, case["train"] / n)] * len(classes)
    if case["biased"]:
        lo, hi = 0.0, 1e3
        for _ in range(60):
            mid = (lo + hi) / 2
            p = [1 - math.exp(-mid * d) for _, d in classes]
            lo, hi = (mid, hi) if sum(c * q for (c, _), q in zip(classes, p)) < case["train"] else (lo, mid)
    sizes, entries = [], []
    L = len(_widths(case)[0])
    for k in range(L + 1):
        sizes.append(sum(c * q for (c, _), q in zip(classes, p)))
        if k < L:
            share = min(1.0, sum(c * d * q for (c, d), q in zip(classes, p)) / nnz)
            entries.append(share * (2.0 * E + n))
            p = [1 - (1 - q) * (1 - share) ** (d - 1) for (_, d), q in zip(classes, p)]
    return 2.0 * E + n, sizes, entries


def work(case):
    """What one pass cannot do without: every input once, every output once (expected sizes of the active sets)."""
    n, op = case["n"], case["op"]
    widths, wide = _widths(case)
    L = len(widths)
    nnz, sizes, entries = _expected_sizes(case)
    by = fl = 0.0
    for l in range(L):
        k = L - l - 1
        F, S, R, path_nnz = widths[l], sizes[k], sizes[k + 1], entries[k]
        if op == "full":
            S = R = float(n)
            path_nnz = nnz
        if op in ("epoch", "full", "backward", "first_epoch", "resume"):
            by += 8 * path_nnz + 8 * R + 4 * F * (S + R)
            fl += 2 * path_nnz * F
        if op in ("combine", "backward"):  # Y and X' read, Y' written on the active rows; both products
            by += 4 * S * (2 * wide[l] + wide[l + 1]) + 8 * wide[l] * wide[l + 1]
            fl += 4 * S * wide[l] * wide[l + 1]
        if op in ("preprocess", "resume"):  # the path's arrays written, or read
            by += 8 * path_nnz + 8 * R
    if op in ("preprocess", "first_epoch"):
        by += 8 * nnz + 4 * n
    return {"bytes": by, "flops": fl}


def tolerance(case):
    if case["op"] == "preprocess":
        return "exact"  # the paths are integers and copied weights
    # 32-bit sums in any order: up to 10^5 terms per row, and the backward loop chains L of them
    return {"rel": 1e-5, "max": 1e-4}
