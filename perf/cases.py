"""Timed cases: what programs that use this library have it do.

A GCN program owns a normalised adjacency operand and multiplies it by dense
feature or gradient matrices. Its calls are:

* ``forward``   the exact aggregation Y = A H through a plan of the static
                operand (every forward pass, every exact backward);
* ``oneoff``    the same product without a plan (one pass over a graph that is
                not kept: mini-batches, inference);
* ``sampled``   the approximated backward product on a cached column slice
                (the steps between two refreshes);
* ``backward``  a refresh step on its own: pair scores, top-k, column slice,
                then the product on the new slice;
* ``random``    the same with the randomized sampler in place of top-k;
* ``train``     a window of ten steps of two-layer GCN training: one refresh
                step with the layer-wise budget allocation, nine sampled ones; then one evaluation pass.

Graphs are seeded stand-ins for the data sets' shapes: power-law (exponent
2.1), near-uniform or Erdos-Renyi degrees, no node locality, symmetric with
self-loops, values 1/sqrt(deg_i deg_j), or the mean aggregator's D^-1 A.
Dense operands are N(0, 1).
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2210_10737_amd as rsc
from paper_2210_10737_amd.gcn import GCN, RscConfig

REFRESH_INTERVAL = 10


def listed():
    return [
        # the smallest graph the benchmark has: 4,096 nodes, mean degree 16,
        # 64 features; one prepared product, bound by latency and launches
        {"name": "tiny_forward", "kind": "forward", "family": "er", "n": 4096, "mean": 16.0, "d": 64},
        # the same graph's backward on a refresh step, half of the columns:
        # a chain of small launches
        {"name": "tiny_backward", "kind": "backward", "family": "er", "n": 4096, "mean": 16.0, "d": 64,
         "budget": 50, "kept": 0.5},
        # a mid-size graph taken once, without a plan, with a feature width
        # that fills no whole vector or cache line
        {"name": "ragged_oneoff", "kind": "oneoff", "family": "powerlaw", "n": 60013, "mean": 27.0, "wmax": 3000.0,
         "d": 41},
        # Yelp-shaped graph, hidden width 512: the first layer's aggregation
        {"name": "yelp_forward", "kind": "forward", "family": "powerlaw", "n": 716847, "mean": 20.0, "wmax": 2000.0,
         "d": 512},
        # the same graph's output layer (100 classes: rows of 400 bytes), the
        # unbiased randomized estimate at half of the columns
        {"name": "yelp_random", "kind": "random", "family": "powerlaw", "n": 716847, "mean": 20.0, "wmax": 2000.0,
         "d": 100, "budget": 50, "kept": 0.35},
        # Reddit-shaped graph: few nodes, rows of hundreds of entries and hubs
        {"name": "reddit_forward", "kind": "forward", "family": "powerlaw", "n": 232965, "mean": 570.0,
         "wmax": 57000.0, "d": 256, "entries": 114.0e6},
        # its cached backward between refreshes, 30 % of the columns
        {"name": "reddit_sampled", "kind": "sampled", "family": "powerlaw", "n": 232965, "mean": 570.0,
         "wmax": 57000.0, "d": 256, "entries": 114.0e6, "budget": 30, "kept": 0.51},
        # ogbn-proteins-shaped graph: every row about 600 entries
        {"name": "proteins_forward", "kind": "forward", "family": "uniform", "n": 132534, "mean": 600.0, "d": 256},
        # its refresh step with the mean aggregator (D^-1 A and its transpose)
        {"name": "proteins_mean_backward", "kind": "backward", "family": "uniform", "n": 132534, "mean": 600.0,
         "d": 256, "budget": 30, "kept": 0.3, "mean_aggr": True},
        # ogbn-products-shaped graph, the largest: exact forward ...
        {"name": "products_forward", "kind": "forward", "family": "powerlaw", "n": 2449029, "mean": 50.0,
         "wmax": 5000.0, "d": 256},
        # ... and its backward on a refresh step, 30 % of the columns
        {"name": "products_backward", "kind": "backward", "family": "powerlaw", "n": 2449029, "mean": 50.0,
         "wmax": 5000.0, "d": 256, "budget": 30, "kept": 0.09},
        # ten training steps of the 300-512-100 network on the Yelp-shaped
        # graph: dense layers, exact forward, allocation, sampled backward
        {"name": "yelp_train", "kind": "train", "family": "powerlaw", "n": 716847, "mean": 20.0, "wmax": 2000.0,
         "d": 512, "in_features": 300, "classes": 100, "budget": 10, "kept": 0.08},
    ]


def draw(rng):
    kind = rng.choice(["forward", "forward", "oneoff", "sampled", "backward", "backward", "random", "train"])
    family = rng.choice(["er", "powerlaw", "powerlaw", "uniform"])
    n = int(math.exp(rng.uniform(math.log(1000), math.log(2449029 if kind != "train" else 400000))))
    top = min(600.0, n / 16.0, (120e6 if kind != "train" else 6e6) / n)
    mean = round(math.exp(rng.uniform(math.log(4.0), math.log(max(top, 5.0)))), 1)
    d = int(math.exp(rng.uniform(math.log(8), math.log(512))))
    if rng.random() < 0.5:
        d = max(8, d // 16 * 16)
    d = min(d, max(8, int(126e6 * 256 / (n * (mean + 1)))))
    case = {"kind": kind, "family": family, "n": n, "mean": mean, "d": d}
    if family == "powerlaw":
        case["wmax"] = round(max(4.0 * mean, min(100.0 * mean, n / 5.0)), 1)
    if kind == "train":
        # the aggregated widths of a network are whole 16-byte vectors
        case.update(d=(d + 3) // 4 * 4, in_features=rng.randrange(32, 300), classes=4 * rng.randrange(2, 28),
                    budget=rng.choice([10, 30]), kept=0.2)
    elif kind in ("sampled", "backward", "random"):
        case["budget"] = rng.choice([10, 20, 30, 50])
        share = case["budget"] / 100.0
        case["kept"] = share if family != "powerlaw" else (0.6 * share if kind == "random" else 0.4 * share)
        if kind != "random" and rng.random() < 0.25:
            case["mean_aggr"] = True
    return case


# ------------------------------------------------------------------ inputs
def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed * 2654435761 % (1 << 62) + 17)
    return g


def _cdf(case, g):
    """Running sum of the nodes' expected degrees. Summed on the host: the
    GPU's scan adds in a varying order, and the last bit can move an edge."""
    n, mean = case["n"], case["mean"]
    if case["family"] == "er":
        w = np.full(n, mean)
    elif case["family"] == "uniform":
        w = mean * (0.75 + 0.5 * torch.rand(n, generator=g, dtype=torch.float64, device="cuda").cpu().numpy())
    else:
        # Pareto with exponent 2.1, cut at wmax; its lower end by bisection on the mean
        a, wmax, lo, hi = 1.1, case["wmax"], 1e-6, mean
        for _ in range(100):
            w0 = 0.5 * (lo + hi)
            cut = (w0 / wmax) ** a
            if w0 * (1.0 - cut ** (1.0 - 1.0 / a)) / (1.0 - 1.0 / a) + cut * wmax < mean:
                lo = w0
            else:
                hi = w0
        w = np.minimum(lo * ((np.arange(n) + 0.5) / n) ** (-1.0 / a), wmax)
    return torch.from_numpy(np.cumsum(w)).cuda()


def _graph(case, seed):
    """(rowptr, col, val) of the symmetric operand on the GPU: endpoints drawn
    by weight, nodes relabelled at random, duplicates and self pairs dropped,
    self-loops added; val are the GCN's, or ones for the mean aggregator."""
    g = _generator(seed)
    n = case["n"]
    cdf = _cdf(case, g)
    label = torch.randperm(n, generator=g, device="cuda")
    m = int(n * case["mean"] / 2)
    ends = []
    for _ in range(2):
        u = torch.rand(m, generator=g, dtype=torch.float64, device="cuda") * cdf[-1]
        ends.append(label[torch.searchsorted(cdf, u).clamp_(max=n - 1)])
        del u
    a, b = torch.minimum(*ends), torch.maximum(*ends)
    del ends
    key = (a * n + b)[a != b]
    del a, b
    key = torch.unique(key)
    i, j = key // n, key % n
    diag = torch.arange(n, device="cuda")
    key = torch.cat([key, j * n + i, diag * n + diag])
    del i, j
    key = torch.sort(key).values
    row, col = key // n, key % n
    del key
    deg = torch.bincount(row, minlength=n)
    rowptr = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    rowptr[1:] = torch.cumsum(deg, 0)
    if case.get("mean_aggr"):
        val = torch.ones(col.numel(), dtype=torch.float32, device="cuda")
    else:
        val = (deg[row].double() * deg[col].double()).rsqrt_().float()
    return rowptr.int(), col.int(), val


def _dense(rows, d, seed):
    """N(0, 1), with the leading dimension rounded up to four floats."""
    ld = (d + 3) // 4 * 4
    return torch.randn((rows, ld), generator=_generator(seed), device="cuda")[:, :d]


def _columns(case):
    return case["n"] * case["budget"] // 100


def _network(case, seed):
    """Features and multi-label targets of the training program."""
    n = case["n"]
    X = torch.randn((n, case["in_features"]), generator=_generator(seed + 1000), device="cuda")
    T = (torch.rand((n, case["classes"]), generator=_generator(seed + 2000), device="cuda") < 0.5).float()
    return X, T


def prepare(case, seed):
    kind = case["kind"]
    rowptr, col, val = _graph(case, seed)
    A = rsc.DeviceCsr(case["n"], case["n"], rowptr, col, val)
    state = {"kind": kind, "step": 0}
    if kind == "train":
        cfg = RscConfig(budget=(case["budget"], 100), refresh_interval=REFRESH_INTERVAL)
        state["model"] = GCN(A, case["in_features"], case["d"], case["classes"], cfg, seed=seed)
        state["X"], state["T"] = _network(case, seed)
        return state
    AT = A
    if case.get("mean_aggr"):
        # the graph is symmetric, so its own arrays are its transpose's
        A, AT = rsc.degree_scale(A), rsc.degree_scale(A, by_column=True, deg_rowptr=rowptr)
    state["A"], state["AT"] = A, AT
    state["B"] = _dense(case["n"], case["d"], seed + 1000)
    if kind == "forward":
        state["plan"] = rsc.SpmmPlan(A)
    elif kind in ("sampled", "backward", "random"):
        state["cache"] = rsc.Cache(AT, A, refresh_interval=REFRESH_INTERVAL)
        state["k"] = _columns(case)
        state["draw_seed"] = seed
        if kind == "sampled":
            # selected at an earlier step, from that step's gradient
            state["cache"].refresh(_dense(case["n"], case["d"], seed + 2000), state["k"], 0)
    return state


def run(state):
    kind = state["kind"]
    if kind == "forward":
        return state["plan"].run(state["B"])
    if kind == "oneoff":
        return rsc.spmm(state["A"], state["B"])
    if kind == "train":
        # the weights stay as they are: the window returns its losses, the
        # gradients its ten backward passes added up and, from the evaluation
        # that closes an epoch, the logits
        model = state["model"]
        model.zero_grad(set_to_none=True)
        losses = [model.train_step(state["X"], state["T"], None, state["step"] + s) for s in range(REFRESH_INTERVAL)]
        state["step"] += REFRESH_INTERVAL
        with torch.no_grad():
            logits = model(state["X"])
        return {"loss": torch.stack([x.detach() for x in losses]), "grad_W1": model.W1.grad,
                "grad_W2": model.W2.grad, "logits": logits}
    cache, B = state["cache"], state["B"]
    if kind == "backward":
        cache.refresh(B, state["k"], state["step"])
        state["step"] += REFRESH_INTERVAL
    elif kind == "random":
        cache.refresh_random(B, state["k"], state["draw_seed"], state["step"])
        state["step"] += REFRESH_INTERVAL
    return cache.spmm_sampled(B)


# -------------------------------------------------------------- the floor
def work(case):
    """Bytes: row pointers, columns and values once, every referenced row of
    the dense operand once, the output once; a refresh reads the operand's
    columns, the kept values and the whole dense operand, writes the slice and
    reads it back. Operations: two per entry and feature."""
    n, d = case["n"], case["d"]
    nnz = case.get("entries", n * (case["mean"] + 1.0))
    dense = 4.0 * n * d
    kind = case["kind"]
    if kind in ("forward", "oneoff"):
        return {"bytes": 4.0 * n + 8.0 * nnz + 2 * dense, "flops": 2.0 * nnz * d}
    kept = case["kept"] * nnz
    if kind == "train":
        # ten steps of dense layers and both layers' aggregations, forward
        # exact, backward on the slices; eleven forward passes
        f, c = case["in_features"], case["classes"]
        gemm = 2.0 * n * (f * d * (11 + 10) + d * c * (11 + 20))
        spmm = 2.0 * (11 * nnz + 10 * kept) * (d + c)
        act = 4.0 * n * (21 * f + 105 * d + 105 * c)
        return {"bytes": act + 16.0 * (11 * nnz + 10 * kept) + 10.0 * nnz, "flops": gemm + spmm}
    product = 4.0 * n + 8.0 * kept + case["budget"] / 100.0 * dense + dense
    refresh = 0.0 if kind == "sampled" else dense + 8.0 * n + 4.0 * nnz + 12.0 * kept
    return {"bytes": product + refresh, "flops": 2.0 * kept * d}


def tolerance(case):
    """fp32 products and short fp32 sums under 64-bit ones: measured 2e-8 to
    1.4e-7 against 64 bits. In training, changing the order of the sums (the
    width of the feature passes) moves the gradients by up to 1.9e-6, because
    values near zero change sides in the ReLU."""
    return {"rel": 8e-6 if case["kind"] == "train" else 6e-7}


# ------------------------------------------------------------- 64-bit truth
def _spmm64(n, rowptr, col, val, B):
    """sum over the entries of each row of val * B[col], in fp64."""
    A = torch.sparse_csr_tensor(rowptr.int(), col.int(), val.double(), size=(n, B.shape[0]), device="cuda")
    return A @ B.double().contiguous()


def _scores64(rowptr, val, B):
    """sqrt of (column square-norm x row square-norm) of every pair; val are
    the values of the transpose, row i of which is column i."""
    n = B.shape[0]
    row = torch.repeat_interleave(torch.arange(n, device="cuda"), (rowptr[1:] - rowptr[:-1]).long())
    cn2 = torch.zeros(n, dtype=torch.float64, device="cuda").index_add_(0, row, val.double() ** 2)
    rn2 = torch.zeros(n, dtype=torch.float64, device="cuda")
    for j in range(B.shape[1]):
        rn2 += B[:, j].double() ** 2
    return (cn2 * rn2).sqrt()


def _draw_scales(p, k, seed):
    """Scale of every column after k draws with replacement, p the scores:
    integer weights, and SplitMix64 (Steele, Lea and Flood 2014) for draw t."""
    w = np.floor(p * (2.0 ** 38 / p.max())).astype(np.int64)
    W = np.cumsum(w)
    t = np.arange(1, k + 1, dtype=np.uint64)
    with np.errstate(over="ignore"):
        z = np.uint64(seed) + t * np.uint64(0x9E3779B97F4A7C15)
        z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
        z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
        z = z ^ (z >> np.uint64(31))
        # floor(z * total / 2^64) from 32-bit halves
        total = int(W[-1])
        lo32 = np.uint64(0xFFFFFFFF)
        z0, z1 = z & lo32, z >> np.uint64(32)
        t0, t1 = np.uint64(total & 0xFFFFFFFF), np.uint64(total >> 32)
        mid = z1 * t0 + ((z0 * t0) >> np.uint64(32))
        mid2 = z0 * t1 + (mid & lo32)
        u = z1 * t1 + (mid >> np.uint64(32)) + (mid2 >> np.uint64(32))
    count = np.bincount(np.searchsorted(W, u.astype(np.int64), side="right"), minlength=len(w))
    return np.where(count > 0, count * float(total) / (float(k) * np.maximum(w, 1)), 0.0)


def exact(case, seed):
    kind, n = case["kind"], case["n"]
    rowptr, col, val = _graph(case, seed)
    if kind == "train":
        # the losses only: the gradients rest on selections made from fp32 gradients
        X, T = _network(case, seed)
        g = torch.Generator().manual_seed(seed)

        def glorot(fan_in, fan_out):
            a = math.sqrt(6.0 / (fan_in + fan_out))
            return ((torch.rand(fan_in, fan_out, generator=g) * 2 - 1) * a).cuda().double()

        W1, W2 = glorot(case["in_features"], case["d"]), glorot(case["d"], case["classes"])
        H1 = torch.relu(_spmm64(n, rowptr, col, val, X.double() @ W1))
        logits = _spmm64(n, rowptr, col, val, H1 @ W2)
        loss = torch.nn.functional.binary_cross_entropy_with_logits(logits, T.double())
        return {"loss": loss.repeat(REFRESH_INTERVAL), "grad_W1": None, "grad_W2": None,
                "logits": logits}
    B = _dense(n, case["d"], seed + 1000)
    deg = (rowptr[1:] - rowptr[:-1]).double()
    valT = val
    if case.get("mean_aggr"):
        row = torch.repeat_interleave(torch.arange(n, device="cuda"), deg.long())
        val, valT = (1.0 / deg[row]).float(), (1.0 / deg[col.long()]).float()
    if kind in ("forward", "oneoff"):
        return _spmm64(n, rowptr, col, val, B)
    scored = _dense(n, case["d"], seed + 2000) if kind == "sampled" else B
    # the backward multiplies by the transpose, whose columns are val's rows
    score = _scores64(rowptr, val, scored)
    k = _columns(case)
    if kind == "random":
        scale = torch.from_numpy(_draw_scales(score.cpu().numpy(), k, seed)).cuda()
        scaled = (valT.double() * scale[col.long()]).float()   # a slice holds fp32 values
        keep = scale[col.long()] > 0
    else:
        kept = torch.zeros(n, dtype=torch.bool, device="cuda")
        kept[torch.sort(score, descending=True, stable=True).indices[:k]] = True
        scaled, keep = valT, kept[col.long()]
    ends = torch.cat([torch.zeros(1, dtype=torch.int64, device="cuda"), torch.cumsum(keep.long(), 0)])
    return _spmm64(n, ends[rowptr.long()], col[keep], scaled[keep], B)
