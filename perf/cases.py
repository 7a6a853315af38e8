"""The work this library is timed on: graph-transformer attention layers and the graph preparation before them.

Six kinds of case, each one call sequence of a training or inference program:

* ``layer``: one sparse attention layer over a prepared graph, forward, or forward and backward;
* ``tiles``: the same at a density threshold low enough that the plan holds dense tiles;
* ``bias``: the same with a per-edge bias (the structural encoding), whose gradient is returned;
* ``full``: one full attention layer (the fully connected layer that is interleaved with the sparse ones);
* ``prepare``: what a program runs once per graph: reorder, relabel, tile plan, and the move of its features.

The graphs are stochastic block models, Chung-Lu power-law graphs and batches of small graphs with a global
token, at the sizes, degrees and feature widths of the repository's workloads.  For the layers the nodes are
already laid out cluster by cluster, a cluster's nodes by falling degree, as the reordering leaves them; for
``prepare`` they are shuffled.  All inputs are made on the GPU from the seed.
"""

import math

import numpy as np
import torch

from paper_2407_14106_amd import gt

DT = {"bf16": torch.bfloat16, "f32": torch.float32}

SBM_100K = dict(graph="sbm", n=100_000, blocks=200, sigma=0.0, degree=16.0, cross=0.15)
SBM_65K = dict(graph="sbm", n=65_536, blocks=256, sigma=0.0, degree=20.0, cross=0.10)
SBM_1M = dict(graph="sbm", n=1_000_000, blocks=1000, sigma=0.5, degree=30.0, cross=0.05)
POWER_1M = dict(graph="power", n=1_000_000, gamma=2.1, degree=12.0, cap=20_000)


def listed():
    return [
        # inference on a small citation-sized graph, one head, fp32: latency and launches
        dict(name="small_f32_forward", kind="layer", graph="sbm", n=4096, blocks=16, sigma=0.0, degree=8.0,
             cross=0.10, heads=1, dim=64, dtype="f32", backward=False),
        # one training step's layer on a batch of 128 molecules with a global token
        dict(name="molecules_step", kind="layer", graph="batch", graphs=128, lo=23, hi=26, degree=2.2,
             heads=8, dim=32, dtype="bf16", backward=True),
        # a layer of node classification at 100K nodes, wide heads
        dict(name="sbm_100k_step", kind="layer", heads=8, dim=64, dtype="bf16", backward=True, **SBM_100K),
        # a million-node power-law graph: hub rows and columns of thousands of edges
        dict(name="power_1m_step", kind="layer", heads=4, dim=32, dtype="bf16", backward=True, **POWER_1M),
        # the headline workload: a million nodes, thirty million edges
        dict(name="sbm_1m_step", kind="layer", heads=8, dim=32, dtype="bf16", backward=True, **SBM_1M),
        # a large batch of molecules: very short rows, and one row and column that hold every node
        dict(name="token_1m_step", kind="layer", graph="batch", graphs=40_000, lo=23, hi=26, degree=2.2,
             heads=8, dim=32, dtype="bf16", backward=True),
        # training in single precision
        dict(name="sbm_65k_f32_step", kind="layer", heads=8, dim=64, dtype="f32", backward=True, **SBM_65K),
        # a clustered graph at the 5% threshold: the densest tiles on the matrix cores, the rest as edges
        dict(name="sbm_65k_tiles_step", kind="tiles", heads=8, dim=64, dtype="bf16", backward=True, tau_ppm=50_000,
             **SBM_65K),
        # a layer with a structural encoding on every edge, trained with the rest
        dict(name="sbm_100k_bias_step", kind="bias", heads=8, dim=64, dtype="bf16", backward=True, **SBM_100K),
        # the interleaved full layer at the largest size of the workloads
        dict(name="full_65k_step", kind="full", n=65_536, heads=8, dim=64, dtype="bf16", backward=True),
        # the full layer over one mid-sized graph, a ragged size
        dict(name="full_3001_step", kind="full", n=3001, heads=8, dim=64, dtype="bf16", backward=True),
        # a power-law graph made ready for training
        dict(name="prepare_power_1m", kind="prepare", heads=4, dim=32, dtype="bf16", **POWER_1M),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_graph(rng, lo, hi, kinds=("sbm", "power", "batch")):
    kind = rng.choice(kinds)
    n = _log(rng, lo, hi)
    if kind == "sbm":
        degree = round(rng.uniform(6, 30), 1)
        return dict(graph="sbm", n=n, blocks=max(1, n // _log(rng, 200, 1200)), sigma=rng.choice([0.0, 0.5]),
                    degree=degree, cross=round(rng.uniform(0.03, 0.2), 3))
    if kind == "power":
        return dict(graph="power", n=n, gamma=round(rng.uniform(2.05, 2.6), 2), degree=round(rng.uniform(6, 16), 1),
                    cap=max(8, n // 50))
    size = _log(rng, 16, min(2000, max(17, n // 2)))
    return dict(graph="batch", graphs=max(1, n // size), lo=max(2, size - size // 8), hi=size + size // 8,
                degree=round(rng.uniform(2.1, 4.6), 2))


def draw(rng):
    kind = rng.choice(["layer"] * 4 + ["full"] * 2 + ["prepare"] * 2 + ["tiles", "bias"])
    heads, dim = rng.choice([1, 2, 4, 8, 8, 16]), rng.choice([32, 64])
    if kind == "full":
        dtype = rng.choice(["bf16", "bf16", "f32"])
        most = 65_536 if dtype == "bf16" else 12_000
        most = min(most, int(most * math.sqrt(512 / (heads * dim))))
        return dict(kind="full", n=_log(rng, 300, most), heads=heads, dim=dim, dtype=dtype,
                    backward=rng.random() < 0.75)
    dtype = rng.choice(["bf16", "bf16", "f32"])
    # at most 1M nodes of 256 features, and fewer where the features are wider
    most = min(1_000_000, 256_000_000 // (heads * dim * (2 if dtype == "f32" else 1)))
    if kind == "prepare":
        return dict(kind="prepare", heads=heads, dim=dim, dtype=dtype, **_draw_graph(rng, 1000, most))
    if kind == "tiles":
        return dict(kind="tiles", heads=heads, dim=dim, dtype=dtype, backward=rng.random() < 0.75,
                    tau_ppm=rng.choice([10_000, 50_000, 100_000]),
                    **_draw_graph(rng, 2000, most // 10, ("sbm", "power")))
    if kind == "bias":
        return dict(kind="bias", heads=heads, dim=dim, dtype=dtype, backward=rng.random() < 0.75,
                    **_draw_graph(rng, 1000, most // 2))
    return dict(kind="layer", heads=heads, dim=dim, dtype=dtype, backward=rng.random() < 0.75,
                **_draw_graph(rng, 1000, most))


# ---------------------------------------------------------------------------------------------- inputs

def _pairs(n, m, fixed, more, uniform):
    """Keys of exactly m distinct node pairs: the fixed ones, and a random choice of those that more(k) draws."""
    keys = torch.empty(0, dtype=torch.int64, device="cuda")
    for _ in range(40):
        if keys.numel() >= m - fixed.numel():
            break
        u, v = more(m - fixed.numel() - keys.numel() + m // 16 + 64)
        new = torch.minimum(u, v) * n + torch.maximum(u, v)
        new = new[(u != v) & ~torch.isin(new, fixed)] if fixed.numel() else new[u != v]
        keys = torch.unique(torch.cat([keys, new]))
    keys = keys[torch.argsort(uniform(keys.numel()))[:m - fixed.numel()]]
    if keys.numel() + fixed.numel() != m:
        raise ValueError("too dense a graph for its size")
    return torch.cat([fixed, keys])


def _csr(n, u, v):
    """Symmetric CSR with self-loops, rows sorted."""
    d = torch.arange(n, device=u.device)
    keys = torch.sort(torch.cat([u * n + v, v * n + u, d * (n + 1)])).values
    rows = torch.div(keys, n, rounding_mode="floor")
    rowptr = torch.zeros(n + 1, dtype=torch.int64, device=u.device)
    torch.cumsum(torch.bincount(rows, minlength=n), 0, out=rowptr[1:])
    return rowptr, (keys - rows * n).to(torch.int32)


def _nodes(case):
    return case["graphs"] * (case["lo"] + case["hi"]) // 2 + 1 if case["graph"] == "batch" else case["n"]


def _n_pairs(case):
    """Undirected edges, the same for every seed (self-loops come on top)."""
    n = _nodes(case)
    if case["graph"] == "batch":  # at least the trees, and the token's edges
        return max(int((n - 1) * case["degree"] / 2), n - 1 - case["graphs"]) + n - 1
    return int(n * case["degree"] / 2)


def _sizes(case, seed):
    """Node count of each block or graph (numpy, small); their sum is the same for every seed."""
    rng = np.random.Generator(np.random.PCG64(seed))
    if case["graph"] == "batch":  # each size as often as any other
        total, span = _nodes(case) - 1, case["hi"] - case["lo"] + 1
        sizes = case["lo"] + np.arange(case["graphs"]) % span
        sizes[0] += total - sizes.sum()
        return rng.permutation(sizes)
    n, nb = case["n"], case["blocks"]
    share = rng.lognormal(0.0, case["sigma"], size=nb) if case["sigma"] else np.ones(nb)
    edges = np.round(np.cumsum(share / share.sum()) * (n - 2 * nb)).astype(np.int64)
    return np.diff(np.concatenate([[0], edges])) + 2


def _graph(case, seed, shuffled):
    """(rowptr, col) on the GPU; nodes cluster by cluster and by falling degree, or shuffled."""
    dev = torch.device("cuda")
    g = torch.Generator(device=dev).manual_seed(seed)
    kind, n, m = case["graph"], _nodes(case), _n_pairs(case)
    none = torch.empty(0, dtype=torch.int64, device=dev)

    def uniform(k):
        return torch.rand(k, generator=g, device=dev, dtype=torch.float64)

    if kind == "power":
        base = torch.arange(1, n + 1, device=dev, dtype=torch.float64) ** (-1.0 / (case["gamma"] - 1.0))
        lo, hi = 0.0, float(case["cap"]) / float(base[-1]) + 1.0
        for _ in range(60):  # the scale at which the capped expected degrees have the asked mean
            mid = 0.5 * (lo + hi)
            lo, hi = (mid, hi) if float(torch.clamp(mid * base, max=case["cap"]).mean()) < case["degree"] else (lo, mid)
        cdf = torch.cumsum(torch.clamp(lo * base, max=case["cap"]), 0)
        cdf = cdf / cdf[-1]
        keys = _pairs(n, m, none, lambda k: tuple(
            torch.searchsorted(cdf, uniform(k), right=True).clamp_(max=n - 1) for _ in range(2)), uniform)
        cluster = torch.zeros(n, dtype=torch.int64, device=dev)
    elif kind == "sbm":
        sizes = torch.from_numpy(_sizes(case, seed)).to(dev)
        nb = sizes.numel()
        starts = torch.cumsum(sizes, 0) - sizes
        weight = torch.cumsum((sizes * (sizes - 1)).double(), 0)

        def more(k):
            cross = int(round(k * case["cross"])) if nb > 1 else 0
            b = torch.searchsorted(weight / weight[-1], uniform(k - cross), right=True).clamp_(max=nb - 1)
            ends = [starts[b] + (uniform(k - cross) * sizes[b]).long() for _ in range(2)]
            return tuple(torch.cat([e, (uniform(cross) * n).long()]) for e in ends)

        keys = _pairs(n, m, none, more, uniform)
        cluster = torch.repeat_interleave(torch.arange(nb, device=dev), sizes)
    else:
        # random trees with a few ring closures, in batch order, and one token (the last node) linked to every node
        sizes = torch.from_numpy(_sizes(case, seed)).to(dev)
        real = n - 1
        starts = torch.cumsum(sizes, 0) - sizes
        of = torch.repeat_interleave(torch.arange(sizes.numel(), device=dev), sizes)
        node = torch.arange(real, device=dev)
        local = node - starts[of]
        parent = starts[of] + (uniform(real) * local).long()
        fixed = torch.cat([(parent * n + node)[local > 0], node * n + real])

        def more(k):
            u = (uniform(k) * real).long()
            return u, starts[of[u]] + (uniform(k) * sizes[of[u]]).long()

        keys = _pairs(n, m, fixed, more, uniform)
        cluster = None
    u = torch.div(keys, n, rounding_mode="floor")
    v = keys - u * n
    if shuffled:
        new = torch.argsort(uniform(n))
    elif cluster is None:
        return _csr(n, u, v)
    else:
        degree = torch.bincount(u, minlength=n) + torch.bincount(v, minlength=n)
        order = torch.argsort(cluster * (m + 1) - degree, stable=True)
        new = torch.empty_like(order)
        new[order] = torch.arange(n, device=dev)
    return _csr(n, new[u], new[v])


def _features(case, n, seed, count):
    g = torch.Generator(device="cuda").manual_seed(seed * 1009 + 7)
    shape = (n, case["heads"], case["dim"])
    return [torch.randn(shape, generator=g, device="cuda").to(DT[case["dtype"]]) for _ in range(count)]


def prepare(case, seed):
    s = {"kind": case["kind"], "backward": case.get("backward", False)}
    if case["kind"] == "full":
        s["x"] = _features(case, case["n"], seed, 4)
        return s
    s["rowptr"], s["col"] = _graph(case, seed, case["kind"] == "prepare")
    n, nnz = s["rowptr"].numel() - 1, s["col"].numel()
    s["x"] = _features(case, n, seed, 1 if case["kind"] == "prepare" else 4)
    if case["kind"] == "prepare":
        return s
    if case["kind"] == "tiles":
        s["plan"] = gt.build_tiles(s["rowptr"], s["col"], 128, case["tau_ppm"])
    elif case["kind"] == "bias":
        s["plan"] = gt.build_tiles(s["rowptr"], s["col"], edge_positions=True)
        s["csc_pos"] = gt.edge_map(s["plan"])
        g = torch.Generator(device="cuda").manual_seed(seed * 1013 + 11)
        s["bias"] = torch.randn((nnz, case["heads"]), generator=g, device="cuda")
    else:
        s["plan"] = gt.build_tiles(s["rowptr"], s["col"])
    return s


# ---------------------------------------------------------------------------------------------- the calls

def run(s):
    if s["kind"] == "prepare":
        perm, iperm, labels = gt.reorder(s["rowptr"], s["col"])
        rowptr, col = gt.permute_csr(s["rowptr"], s["col"], perm, iperm)
        plan = gt.build_tiles(rowptr, col)
        x = gt.gather_rows(s["x"][0], perm)
        # the plan's arrays whose sizes follow from the graph's, and its two edge lists padded to the graph's edges
        a = plan.arrays
        edges = {k: torch.nn.functional.pad(a[k], (0, col.numel() - a[k].numel()), value=-1)
                 for k in ("sp_col", "sp_row")}
        return {"perm": perm, "iperm": iperm, "labels": labels, "rowptr": rowptr, "col": col, "x": x, **edges,
                **{k: a[k] for k in ("tile_rowptr", "sp_rowptr", "sp_colptr", "tileT_ptr")}}
    Q, K, V, dO = s["x"]
    if s["kind"] == "full":
        O, L = gt.dense_attn_fwd(Q, K, V)
        return (O, L, *gt.dense_attn_bwd(Q, K, V, O, dO, L)) if s["backward"] else (O, L)
    if s["kind"] == "bias":
        O, L = gt.sparse_attn_fwd_bias(s["plan"], Q, K, V, s["bias"])
        if not s["backward"]:
            return O, L
        return (O, L, *gt.sparse_attn_bwd_bias(s["plan"], s["csc_pos"], Q, K, V, s["bias"], dO, L))
    O, L = gt.sparse_attn_fwd(s["plan"], Q, K, V)
    return (O, L, *gt.sparse_attn_bwd(s["plan"], Q, K, V, dO, L)) if s["backward"] else (O, L)


# ---------------------------------------------------------------------------------------------- what it takes

def work(case):
    """Bytes and operations of one pass: every input and output once."""
    item = 2 if case["dtype"] == "bf16" else 4
    width = case["heads"] * case["dim"]
    back = case.get("backward", False)
    n = case["n"] if case["kind"] == "full" else _nodes(case)
    if case["kind"] == "full":
        features = n * width * item * (8 if back else 4) + n * case["heads"] * 4
        return {"bytes": features, "flops": n * n * width * (14 if back else 4)}
    nnz = 2 * _n_pairs(case) + n
    csr = 8 * (n + 1) + 4 * nnz
    if case["kind"] == "prepare":
        # the CSR in; the relabelled CSR, both orders of the plan's edges, three node arrays and the moved rows out
        return {"bytes": 2 * csr + 2 * csr + 12 * n + 2 * n * width * item, "flops": nnz}
    features = n * width * item * (8 if back else 4) + n * case["heads"] * 4
    bias = 4 * nnz * case["heads"] * (2 if back else 1) if case["kind"] == "bias" else 0
    return {"bytes": csr + features + bias, "flops": nnz * width * (14 if back else 4)}


def tolerance(case):
    """About four times the largest error against 64 bits: 2.4e-3 in bf16; in fp32 2.5e-7 over a node's edges, and
    1.7e-6 over all nodes of a full layer (whose outputs are means of thousands of values that cancel)."""
    if case["kind"] == "prepare":
        return "exact"
    if case["dtype"] == "bf16":
        return {"rel": 1e-2, "max": 0.1}
    return {"rel": 8e-6, "max": 1e-3} if case["kind"] == "full" else {"rel": 2e-6, "max": 2e-4}


def exact(case, seed):
    """What run() returns, in 64 bits (nothing for `prepare`, whose outputs are whole numbers)."""
    if case["kind"] == "prepare":
        return None
    if case["kind"] == "full":
        return _exact_full(_features(case, case["n"], seed, 4), case.get("backward", False))
    rowptr, col = _graph(case, seed, False)
    n, nnz = rowptr.numel() - 1, col.numel()
    x = _features(case, n, seed, 4)
    bias = None
    if case["kind"] == "bias":
        g = torch.Generator(device="cuda").manual_seed(seed * 1013 + 11)
        bias = torch.randn((nnz, case["heads"]), generator=g, device="cuda")
    return _exact_sparse(rowptr, col, x, bias, case["backward"])


def _exact_sparse(rowptr, col, x, bias, backward):
    Q, K, V, dO = x
    n, H, d = Q.shape
    scale = 1.0 / math.sqrt(d)
    dev, nnz = col.device, col.numel()
    col = col.long()
    row = torch.repeat_interleave(torch.arange(n, device=dev), rowptr[1:] - rowptr[:-1])
    step = max(1, (1 << 28) // (H * d))  # edges at a time: 2 GiB of products
    parts = [slice(a, min(nnz, a + step)) for a in range(0, nnz, step)]

    def dots(A, B):
        out = torch.empty((nnz, H), dtype=torch.float64, device=dev)
        for p in parts:
            out[p] = (A[row[p]].double() * B[col[p]].double()).sum(-1)
        return out

    def order_by(ids):
        """The edges in the order of ids, the piece of up to 256 edges of one id each belongs to, the pieces' ids."""
        order = torch.argsort(ids, stable=True)
        ptr = torch.zeros(n + 1, dtype=torch.int64, device=dev)
        torch.cumsum(torch.bincount(ids, minlength=n), 0, out=ptr[1:])
        pieces = torch.div(ptr[1:] - ptr[:-1] + 255, 256, rounding_mode="floor")
        first = torch.cumsum(pieces, 0) - pieces
        ids = ids[order]
        at = torch.arange(nnz, device=dev) - ptr[ids]
        piece = first[ids] + torch.div(at, 256, rounding_mode="floor")
        return order, piece, torch.repeat_interleave(torch.arange(n, device=dev), pieces)

    def summed(by, value, *shape):
        """Sum of value(edges) over the edges of each id, piece by piece (an id may hold every edge)."""
        order, piece, of = by
        table = torch.zeros((of.numel(), *shape), dtype=torch.float64, device=dev)
        for p in parts:
            table.index_add_(0, piece[p], value(order[p]))
        return torch.zeros((n, *shape), dtype=torch.float64, device=dev).index_add_(0, of, table)

    rows, cols = order_by(row), order_by(col)
    w = dots(Q, K).mul_(scale)
    if bias is not None:
        w += bias.double()
    w.exp_()  # scores of normal draws stay far below the range of the 64-bit exponential
    total = summed(rows, lambda e: w[e], H)
    P = w / total[row]
    del w
    O = summed(rows, lambda e: P[e].unsqueeze(-1) * V[col[e]].double(), H, d)
    if not backward:
        return O, torch.log(total)
    dP = dots(dO, V)
    D = summed(rows, lambda e: P[e] * dP[e], H)
    dS = dP.sub_(D[row]).mul_(P)
    grads = [summed(rows, lambda e: dS[e].unsqueeze(-1) * K[col[e]].double(), H, d).mul_(scale),
             summed(cols, lambda e: dS[e].unsqueeze(-1) * Q[row[e]].double(), H, d).mul_(scale),
             summed(cols, lambda e: P[e].unsqueeze(-1) * dO[row[e]].double(), H, d)]
    return (O, torch.log(total), *grads) if bias is None else (O, torch.log(total), *grads, dS)


def _exact_full(x, backward):
    Q, K, V, dO = x
    n, H, d = Q.shape
    scale = 1.0 / math.sqrt(d)
    out = [torch.zeros((n, H, d), dtype=torch.float64, device=Q.device) for _ in range(4 if backward else 1)]
    lse = torch.empty((n, H), dtype=torch.float64, device=Q.device)
    step = max(1, (1 << 28) // n)  # rows at a time: 2 GiB of scores
    for h in range(H):
        q, k, v, g = (t[:, h].double().contiguous() for t in x)
        kt, vt = k.t().contiguous(), v.t().contiguous()
        for a in range(0, n, step):
            p = slice(a, min(n, a + step))
            s = torch.mm(q[p], kt).mul_(scale)
            lse[p, h] = torch.logsumexp(s, 1)
            s.sub_(lse[p, h].unsqueeze(1)).exp_()
            out[0][p, h] = torch.mm(s, v)
            if backward:
                out[3][:, h] += torch.mm(s.t(), g[p])
                ds = torch.mm(g[p], vt)
                ds.sub_((g[p] * out[0][p, h]).sum(1, keepdim=True)).mul_(s)
                out[1][p, h] = torch.mm(ds, k) * scale
                out[2][:, h] += torch.mm(ds.t(), q[p]) * scale
    return (out[0], lse, *out[1:])
