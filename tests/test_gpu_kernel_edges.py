"""GPU attention at the sizes where the kernels' loops and dispatch rules change:
row and column lengths around the id chunks and the long-row cut, few and many
long rows and their folded runs, rows without edges beside infinite features,
the full layer's workgroup shapes, and tile plans of every chunk-plan size."""

import numpy as np
import pytest
import torch

from oracle import attention as OA
from synth import csr_from_pairs
from synth.tensors import normal_tensor
from tests.helpers import assert_close, dev_csr, dev_feat, host
from tests.test_gpu_attention import CSR_ONLY, feats, run_case, say
from tests.test_gpu_bias import run_bias_case

pytestmark = pytest.mark.gpu


def both_ways(degs, m, seed):
    """2 m nodes: node r < m attends to degs[r] of the nodes from m on, and node m + r is attended by degs[r]
    of the nodes below m (columns beyond the first len(degs) rows' own picks), so rows and columns have the given
    lengths where nothing else was drawn."""
    rng = np.random.default_rng(seed)
    u, v = [], []
    for r, d in enumerate(degs):
        u.append(np.full(d, r))
        v.append(m + rng.choice(m, size=d, replace=False))
        u.append(m + rng.choice(m, size=d, replace=False))
        v.append(np.full(d, r))
    return csr_from_pairs(2 * m, np.concatenate(u), np.concatenate(v), symmetric=False, self_loops=False)


# around the id chunks of 2 to 64 entries, the edges taken at a time, the long-row cut (256) and the runs of 32
DEGREES = list(range(0, 36)) + [47, 48, 49, 63, 64, 65, 127, 128, 129, 255, 256, 257, 287, 288, 289, 320, 513]


@pytest.mark.parametrize("dtype,H,d", [("f32", 1, 32), ("f32", 8, 64), ("f32", 16, 64), ("bf16", 1, 32),
                                       ("bf16", 4, 32), ("bf16", 8, 32), ("bf16", 8, 64), ("bf16", 16, 64)])
def test_row_and_column_lengths(gt, dtype, H, d):
    rowptr, col = both_ways(DEGREES, 520, H + d)
    deg = np.diff(rowptr)
    assert np.array_equal(deg[:len(DEGREES)], DEGREES)
    assert np.array_equal(np.bincount(col, minlength=1040)[:len(DEGREES)], DEGREES)
    run_case(gt, rowptr, col, H, d, dtype, taus=(CSR_ONLY,), seed=11)


@pytest.mark.parametrize("n_long,length", [(1, 16_500), (64, 260), (65, 260), (130, 257), (2, 9_000),
                                           (1025, 257), (2049, 257)])
def test_long_row_lists(gt, n_long, length):
    # lists of one wavefront and beyond (their runs planned on the device), with the runs folded (more than
    # 16,384 remainder edges) before the merge or, over 2,048 rows, not; over 1,024 rows take the planning workgroup
    # a second round
    degs = [length + (r % 3) for r in range(n_long)] + [0, 1, 5]
    rowptr, col = both_ways(degs, max(length + 3, 600, n_long + 3), n_long)
    assert len(col) > 16_384
    run_case(gt, rowptr, col, 2, 32, "bf16", taus=(CSR_ONLY,), seed=n_long)
    # fp32 where the rows hold 28 edges and more: a row of one edge has dS = dP - D = 0, and what is left is the
    # rounding of its terms (2^-24 scale |dO| |V| |K|, about 1e-6 for d = 64), above 1e-5 of a result that is zero
    # in all rows but one
    if n_long in (65, 130):
        run_case(gt, rowptr, col, 1, 64, "f32", taus=(CSR_ONLY,), seed=n_long)


@pytest.mark.parametrize("n_long", [8192, 8193])
def test_long_row_lists_planned_by_many_workgroups(gt, n_long):
    # rows of 257 and 258 partners among 300 nodes, which attend to themselves: every output is the partners' mean, as
    # every key is the same (weights of 2^-8 relative error in bf16, 300 values of size 1)
    rng = np.random.default_rng(n_long)
    n = n_long + 300
    deg = np.concatenate([257 + np.arange(n_long) % 2, np.ones(300, np.int64)])
    rowptr = np.concatenate([[0], np.cumsum(deg)])
    first = rng.integers(0, 300 - 258, size=n_long)
    col = np.concatenate([(n_long + first[:, None] + np.arange(258))[np.arange(258) < deg[:n_long, None]],
                          n_long + np.arange(300)])
    q, k, v, _ = feats(n, 1, 32, "bf16", 3)
    k[:] = k[:1]
    plan = gt.build_tiles(*dev_csr(rowptr, col), 128, CSR_ONLY)
    O, L = gt.sparse_attn_fwd(plan, *(dev_feat(x, "bf16") for x in (q, k, v)), 0.25)
    torch.cuda.synchronize()
    sums = np.concatenate([np.zeros((1, 1, 32)), np.cumsum(np.asarray(v[n_long:], np.float64), axis=0)])
    a = np.concatenate([first, np.arange(300)])
    assert_close(host(O), (sums[a + deg] - sums[a]) / deg[:, None, None], "bf16", "O")
    s = 0.25 * np.einsum("nhc,hc->nh", np.asarray(q, np.float64), np.asarray(k[0], np.float64))
    assert_close(L.cpu().numpy(), s + np.log(deg)[:, None], "bf16", "LSE")


@pytest.mark.parametrize("dtype,H,d", [("f32", 1, 64), ("f32", 8, 64), ("bf16", 1, 32), ("bf16", 8, 32),
                                       ("bf16", 8, 64)])
def test_bias_row_and_column_lengths(gt, dtype, H, d):
    # the positions' chunks and the quads at every row length; the positions read from the plan, then taken from the
    # list position
    rowptr, col = both_ways(DEGREES, 520, H + d)
    run_bias_case(gt, rowptr, col, H, d, dtype, seed=12)
    rp, cl = dev_csr(rowptr, col)
    arrays = [dev_feat(x, dtype) for x in feats(len(rowptr) - 1, H, d, dtype, 13)]
    B = torch.from_numpy(np.random.default_rng(4).normal(size=(len(col), H)).astype(np.float32)).cuda()
    outs = []
    for positions in (True, False):
        plan = gt.build_tiles(rp, cl, 128, CSR_ONLY, edge_positions=positions)
        O, L = gt.sparse_attn_fwd_bias(plan, *arrays[:3], B)
        outs.append((O, L, *gt.sparse_attn_bwd_bias(plan, gt.edge_map(plan), *arrays[:3], B, arrays[3], L)))
    torch.cuda.synchronize()
    for name, a, b in zip(("O", "LSE", "dQ", "dK", "dV", "dB"), *outs):
        assert torch.equal(a, b), name


@pytest.mark.parametrize("dtype,H,d", [("bf16", 2, 32), ("f32", 1, 64)])
def test_bias_on_many_long_rows(gt, dtype, H, d):
    # 65 long rows and columns: their runs are planned on the device
    rowptr, col = both_ways([260 + (r % 3) for r in range(65)] + [0, 2, 5], 600, 65)
    run_bias_case(gt, rowptr, col, H, d, dtype, seed=14)


@pytest.mark.parametrize("H,d", [(1, 32), (8, 64)])
def test_long_rows_sum_in_short_chains(gt, H, d):
    # 9M edges of long rows, equal weights and equal partners, so that every addition of a run rounds the same way.
    # No serial chain is longer than that of the longest short row, 256 edges: its k-th sum errs by 2^-24 k / 256
    # of the result at most, 128 2^-24 in all; the merge of a row's 94 runs or fewer, the sum of the weights, exp2 and
    # log add less than 30 (a run of 2,208 edges gave 390).
    n = 3000
    Q = torch.zeros(n, H, d, device="cuda")
    x = torch.from_numpy(np.random.default_rng(1).uniform(1, 2, size=(1, H, d)).astype(np.float32)).cuda()
    X = x.expand(n, H, d).contiguous()
    plan = gt.build_tiles(torch.arange(n + 1, dtype=torch.int64, device="cuda") * n,
                          torch.arange(n, dtype=torch.int32, device="cuda").repeat(n), 128, CSR_ONLY)
    O, L = gt.sparse_attn_fwd(plan, Q, X, X, 1.0)
    dV = gt.sparse_attn_bwd(plan, Q, X, X, X, L, 1.0)[2]
    torch.cuda.synchronize()
    for name, a in (("O", O), ("dV", dV)):
        err = float((a.double() / X.double() - 1).abs().max()) * 2 ** 24
        assert err <= 158, (name, err)


@pytest.mark.parametrize("n", [16_384, 32_767, 32_768, 33_001])
def test_node_runs_over_the_dies(gt, n):
    # from some size on each die walks runs of the node range: every node exactly once
    rng = np.random.default_rng(n)
    u = rng.integers(0, n, size=2 * n)
    v = (u + rng.integers(-40, 41, size=2 * n)) % n
    rowptr, col = csr_from_pairs(n, u, v, symmetric=False, self_loops=True)
    run_case(gt, rowptr, col, 8, 32, "bf16", taus=(CSR_ONLY,), seed=n)


@pytest.mark.parametrize("dtype,H,d", [("f32", 2, 32), ("bf16", 1, 32), ("bf16", 8, 64)])
def test_infinite_features_stay_with_their_edges(gt, dtype, H, d):
    # The last node x (which ends the edge list) holds infinities; it attends to itself and node 1, and only node 2
    # attends to it.  Every other row, with edges or without, and every other column is as with finite features.
    n, x = 203, 202
    rng = np.random.default_rng(7)
    u = np.concatenate([rng.integers(3, 150, size=700), [2, x, x]])
    v = np.concatenate([rng.integers(3, 200, size=700), [x, 1, x]])
    rowptr, col = csr_from_pairs(n, u, v, symmetric=False, self_loops=False)
    rp, cl = dev_csr(rowptr, col)
    plan = gt.build_tiles(rp, cl, 64, CSR_ONLY)
    outs = []
    for value in (0.5, np.inf):
        arrays = feats(n, H, d, dtype, 5)
        for a in arrays:
            a[x] = value
        Q, K, V, dO = (dev_feat(a, dtype) for a in arrays)
        O, L = gt.sparse_attn_fwd(plan, Q, K, V, 0.25)
        dQ, dK, dV = gt.sparse_attn_bwd(plan, Q, K, V, dO, L, 0.25)
        torch.cuda.synchronize()
        outs.append((O, L, dQ, dK, dV))
    for k, name in enumerate(("O", "LSE", "dQ", "dK", "dV")):
        keep = torch.ones(n, dtype=torch.bool, device="cuda")
        keep[[2, x] if k < 3 else [1, x]] = False
        a, b = outs[0][k][keep], outs[1][k][keep]
        assert torch.equal(a, b), name
        assert k == 1 or bool(torch.isfinite(a).all()), name


@pytest.mark.parametrize("n,H,d", [(1, 2, 32), (31, 2, 64), (32, 1, 32), (33, 1, 32), (64, 16, 64), (65, 4, 32),
                                   (1025, 16, 32), (2047, 16, 64), (2049, 16, 32), (4065, 8, 64), (4097, 16, 32)])
def test_full_layer_shapes(gt, n, H, d):
    # up to 128, 256, 512 and more workgroups of 128 rows; the keys grow by powers of two along the partners (exact
    # in bf16), so the rows' maxima move late in the walk.  Weights are rounded to 8 bits: |error of O| <= 2^-8 max |v|
    # <= 0.02 for these normals, the tolerance's floor.
    say("full", n, H, d)
    q, k, v, do = (normal_tensor((n, H, d), (n, H, d, t), "bf16") for t in range(4))
    scale = 1.0 / np.sqrt(d)
    Q, K, V, dO = (dev_feat(a, "bf16") for a in (q, k, v, do))
    grown = k * (2.0 ** (4 * np.arange(n) // n))[:, None, None].astype(k.dtype)
    O, L = gt.dense_attn_fwd(Q, dev_feat(grown, "bf16"), V, scale)
    O_ref, L_ref = OA.dense_attn_fwd(q, grown, v, scale)
    assert_close(host(O), O_ref, "bf16", "O, growing keys")
    assert_close(L.cpu().numpy(), L_ref, "bf16", "LSE, growing keys")
    O, L = gt.dense_attn_fwd(Q, K, V, scale)
    dQ, dK, dV = gt.dense_attn_bwd(Q, K, V, O, dO, L, scale)
    torch.cuda.synchronize()
    O_ref, L_ref = OA.dense_attn_fwd(q, k, v, scale)
    assert_close(host(O), O_ref, "bf16", "O")
    assert_close(L.cpu().numpy(), L_ref, "bf16", "LSE")
    for name, a, r in zip(("dQ", "dK", "dV"), (dQ, dK, dV), OA.dense_attn_bwd(q, k, v, do, scale)):
        assert_close(host(a), r, "bf16", name)


@pytest.mark.parametrize("R", [1024, 1025, 4097, 8193])
def test_tile_plans_of_every_size(gt, R):
    # six dense tiles (more than one chunk) in tile rows and tile columns at both ends of the plan and of its
    # rounds of 64 and 1,024 rows; one node in the last tile row
    T = 64
    n = T * (R - 1) + 1
    rng = np.random.default_rng(R)
    u, v = [np.arange(n)], [np.arange(n)]
    for I in sorted({0, 63, 64, 1023, 1024, R - 2} & set(range(R - 1))):
        for J in range(2, 8):
            a, b = I * T + rng.integers(0, T, size=900), J * T + rng.integers(0, T, size=900)
            u += [a, b]
            v += [b, a]
    rowptr, col = csr_from_pairs(n, np.concatenate(u), np.concatenate(v), symmetric=False, self_loops=False)
    run_case(gt, rowptr, col, 1, 32, "bf16", taus=(100_000,), T=T, seed=R)


@pytest.mark.parametrize("scale", [-0.2, 0.0])
@pytest.mark.parametrize("n,H,d,dtype", [(33, 1, 32, "bf16"), (64, 2, 64, "bf16"), (1025, 4, 64, "bf16"),
                                         (4097, 16, 32, "bf16"), (300, 2, 32, "f32")])
def test_full_layer_scale_of_either_sign(gt, n, H, d, dtype, scale):
    # a scale that is not positive leaves the partners past the end (n is ragged for the stages of 64) without weight
    say("full", n, H, d, dtype, scale)
    q, k, v, do = (normal_tensor((n, H, d), (n, H, d, t), dtype) for t in range(4))
    Q, K, V, dO = (dev_feat(a, dtype) for a in (q, k, v, do))
    O, L = gt.dense_attn_fwd(Q, K, V, scale)
    dQ, dK, dV = gt.dense_attn_bwd(Q, K, V, O, dO, L, scale)
    torch.cuda.synchronize()
    O_ref, L_ref = OA.dense_attn_fwd(q, k, v, scale)
    assert_close(host(O), O_ref, dtype, "O")
    assert_close(L.cpu().numpy(), L_ref, dtype, "LSE")
    for name, a, r in zip(("dQ", "dK", "dV"), (dQ, dK, dV), OA.dense_attn_bwd(q, k, v, do, scale)):
        assert_close(host(a), r, dtype, name)


@pytest.mark.parametrize("scale", [-0.2, 0.0])
@pytest.mark.parametrize("T", [64, 128])
def test_dense_tiles_scale_of_either_sign(gt, T, scale):
    # every non-empty tile dense, most of its pairs masked, and none
    rng = np.random.default_rng(T)
    n, H, d = 203, 2, 32
    rowptr, col = csr_from_pairs(n, rng.integers(0, n, size=1500), rng.integers(0, n, size=1500), symmetric=False,
                                 self_loops=False)
    q, k, v, do = feats(n, H, d, "bf16", T)
    Q, K, V, dO = (dev_feat(a, "bf16") for a in (q, k, v, do))
    O_ref, L_ref = OA.sparse_attn_fwd(rowptr, col, q, k, v, scale)
    ref = OA.sparse_attn_bwd(rowptr, col, q, k, v, do, scale)
    for tau in (0, CSR_ONLY):
        plan = gt.build_tiles(*dev_csr(rowptr, col), T, tau)
        O, L = gt.sparse_attn_fwd(plan, Q, K, V, scale)
        dQ, dK, dV = gt.sparse_attn_bwd(plan, Q, K, V, dO, L, scale)
        torch.cuda.synchronize()
        assert_close(host(O), O_ref, "bf16", f"O tau={tau}")
        assert_close(L.cpu().numpy(), L_ref, "bf16", f"LSE tau={tau}")
        for name, a, r in zip(("dQ", "dK", "dV"), (dQ, dK, dV), ref):
            assert_close(host(a), r, "bf16", f"{name} tau={tau}")


@pytest.mark.parametrize("n,H,d", [(33, 2, 64), (97, 1, 32), (1025, 4, 64), (4097, 16, 32)])
def test_full_layer_infinite_last_node(gt, n, H, d):
    # one infinite feature of the last node's V (dO): that feature of every O (dV) row is infinite, every weight being
    # positive, and all other features are those of the finite layer bit for bit
    q, k, v, do = (normal_tensor((n, H, d), (n, H, d, t), "bf16") for t in range(4))
    scale, f = 1.0 / np.sqrt(d), 5
    Q, K = dev_feat(q, "bf16"), dev_feat(k, "bf16")
    outs = []
    for value in (0.5, np.inf):
        v[-1, :, f] = do[-1, :, f] = value
        V, dO = dev_feat(v, "bf16"), dev_feat(do, "bf16")
        O, L = gt.dense_attn_fwd(Q, K, V, scale)
        if not outs:
            O_finite = O
        dV = gt.dense_attn_bwd(Q, K, V, O_finite, dO, L, scale)[2]
        torch.cuda.synchronize()
        outs.append((O, L, dV))
    assert torch.equal(outs[0][1], outs[1][1])
    for k_, name in ((0, "O"), (2, "dV")):
        a, b = outs[0][k_], outs[1][k_]
        assert bool((b[:, :, f] == np.inf).all()), name
        rest = [x for x in range(d) if x != f]
        assert torch.equal(a[:, :, rest], b[:, :, rest]), name


@pytest.mark.parametrize("n,T", [(70, 64), (129, 128), (200, 128)])
def test_dense_tiles_infinite_last_node(gt, n, T):
    # as above for O on dense tiles: every pair is an edge, the last tiles hold columns past the end
    H, d, f = 2, 64, 5
    rowptr, col = csr_from_pairs(n, np.repeat(np.arange(n), n), np.tile(np.arange(n), n), symmetric=False,
                                 self_loops=False)
    plan = gt.build_tiles(*dev_csr(rowptr, col), T, 0)
    assert plan.nnz_sparse == 0
    q, k, v, _ = feats(n, H, d, "bf16", n)
    outs = []
    for value in (0.5, np.inf):
        v[-1, :, f] = value
        outs.append(gt.sparse_attn_fwd(plan, *(dev_feat(x, "bf16") for x in (q, k, v)), 0.125)[0])
    torch.cuda.synchronize()
    assert bool((outs[1][:, :, f] == np.inf).all())
    rest = [x for x in range(d) if x != f]
    assert torch.equal(outs[0][:, :, rest], outs[1][:, :, rest])


@pytest.mark.parametrize("dtype,H,d", [("f32", 2, 32), ("f32", 8, 64), ("bf16", 1, 32), ("bf16", 8, 32)])
def test_bias_near_the_lowest_value(gt, dtype, H, d):
    # A row whose every score is one large negative finite number (-2.2e38: -3.17e38 in the exp2 domain, where it
    # absorbs the scaled product) takes the mean of its partners; beside finite scores the same bias gives no weight.
    # Rows of 1 edge, of a few, around the long-row cut, and long.
    degs = [1, 2, 3, 31, 255, 256, 257, 700]
    m = len(degs)
    rowptr, col = both_ways(degs + degs, 720, H + d)
    n, nnz, low = len(rowptr) - 1, len(col), -2.2e38
    q, k, v, _ = feats(n, H, d, dtype, 21)
    bias = np.random.default_rng(3).normal(size=(nnz, H)).astype(np.float32)
    for r in range(2 * m):
        a, b = rowptr[r], rowptr[r + 1]
        bias[a:b if r < m else a + (b - a) // 2] = low
    plan = gt.build_tiles(*dev_csr(rowptr, col), 64, CSR_ONLY)
    O, L = gt.sparse_attn_fwd_bias(plan, *(dev_feat(x, dtype) for x in (q, k, v)), torch.from_numpy(bias).cuda(), 0.25)
    torch.cuda.synchronize()
    # the same rows with equal scores of ordinary size (in 64 bits too, the low score would absorb log l of the LSE)
    bias[:rowptr[m]] = 0
    q[:m] = 0
    O_ref, L_ref = OA.sparse_attn_fwd(rowptr, col, q, k, v, 0.25, bias=bias)
    L_ref[:m] = low
    assert_close(host(O), O_ref, dtype, "O")
    assert_close(L.cpu().numpy(), L_ref, dtype, "LSE")


def shifted(x, off):
    """The same tensor as a contiguous view `off` elements into a larger buffer."""
    buf = torch.empty(x.numel() + 16, dtype=x.dtype, device=x.device)
    out = buf[off:off + x.numel()].view(x.shape)
    out.copy_(x)
    assert out.is_contiguous() and out.data_ptr() % 16 == off * x.element_size() % 16
    return out


# which of Q, K, V, dO lie at which offset (elements; 8 are 16 bytes)
OFFSETS = [(1, 1, 1, 1), (4, 4, 4, 4), (8, 8, 8, 8), (1, 0, 0, 0), (0, 4, 0, 0), (0, 0, 2, 0), (0, 0, 0, 1)]


@pytest.mark.parametrize("offs", OFFSETS)
@pytest.mark.parametrize("n,H,d", [(129, 2, 32), (300, 4, 64)])
def test_full_layer_features_at_any_address(gt, n, H, d, offs):
    arrays = [normal_tensor((n, H, d), (n, H, d, t), "bf16") for t in range(4)]
    scale = 1.0 / np.sqrt(d)
    Q, K, V, dO = (shifted(dev_feat(x, "bf16"), off) for x, off in zip(arrays, offs))
    O, L = gt.dense_attn_fwd(Q, K, V, scale)
    dQ, dK, dV = gt.dense_attn_bwd(Q, K, V, O, dO, L, scale)
    torch.cuda.synchronize()
    O_ref, L_ref = OA.dense_attn_fwd(*arrays[:3], scale)
    assert_close(host(O), O_ref, "bf16", "O")
    assert_close(L.cpu().numpy(), L_ref, "bf16", "LSE")
    for name, a, r in zip(("dQ", "dK", "dV"), (dQ, dK, dV), OA.dense_attn_bwd(*arrays, scale)):
        assert_close(host(a), r, "bf16", name)


@pytest.mark.parametrize("offs", OFFSETS)
@pytest.mark.parametrize("T,tau,H,d", [(64, 0, 2, 64), (128, 0, 4, 32), (128, CSR_ONLY, 8, 32)])
def test_sparse_layer_features_at_any_address(gt, T, tau, H, d, offs):
    # every non-empty tile dense, or none; without and with a bias
    n, scale = 203, 0.2
    rng = np.random.default_rng(T + H)
    rowptr, col = csr_from_pairs(n, rng.integers(0, n, size=3000), rng.integers(0, n, size=3000), symmetric=False,
                                 self_loops=True)
    arrays = feats(n, H, d, "bf16", T)
    bias = rng.normal(size=(len(col), H)).astype(np.float32)
    plan = gt.build_tiles(*dev_csr(rowptr, col), T, tau, edge_positions=True)
    B = torch.from_numpy(bias).cuda()
    Q, K, V, dO = (shifted(dev_feat(x, "bf16"), off) for x, off in zip(arrays, offs))
    for b in (None, bias):
        if b is None:
            O, L = gt.sparse_attn_fwd(plan, Q, K, V, scale)
            grads = gt.sparse_attn_bwd(plan, Q, K, V, dO, L, scale)
        else:
            O, L = gt.sparse_attn_fwd_bias(plan, Q, K, V, B, scale)
            grads = gt.sparse_attn_bwd_bias(plan, gt.edge_map(plan), Q, K, V, B, dO, L, scale)
        torch.cuda.synchronize()
        O_ref, L_ref = OA.sparse_attn_fwd(rowptr, col, *arrays[:3], scale, bias=b)
        assert_close(host(O), O_ref, "bf16", "O")
        assert_close(L.cpu().numpy(), L_ref, "bf16", "LSE")
        ref = OA.sparse_attn_bwd(rowptr, col, *arrays, scale, bias=b)
        for name, a, r in zip(("dQ", "dK", "dV", "dB"), grads, ref):
            assert_close(host(a), r, "bf16", name)
