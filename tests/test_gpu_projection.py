"""GPU parity of the projection with bisection (Section 3.4, Algorithm 1 of arXiv 2109.00170):
block scores, top-N selection and the bisection against the oracle - integer and index work, so
everything is compared bit for bit (scores included: their arithmetic order is part of the
definition)."""
import ctypes

import numpy as np
import pytest

import oracle
import paper_2109_00170_amd as alcs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Cout,Cin,k,V", [(8, 5, 1, 4), (10, 3, 3, 4), (7, 4, 1, 2), (33, 2, 3, 16), (5, 5, 1, 1),
                                          (64, 129, 1, 8), (256, 257, 1, 4), (30, 64, 3, 4)])
def test_block_scores_bit_exact(Cout, Cin, k, V):
    import torch
    rng = np.random.default_rng(3000 + Cout + Cin)
    W = (rng.standard_normal((Cout, Cin, k, k)) * rng.random((Cout, 1, 1, 1)) * 3).astype(np.float32)
    W[rng.random(W.shape) < 0.1] = 0
    got = alcs.alcs_block_scores(torch.from_numpy(W).cuda(), V)
    torch.cuda.synchronize()
    want = oracle.block_scores(W, V)
    assert got.cpu().numpy().tobytes() == want.tobytes()


def scores_with_ties(n, seed):
    rng = np.random.default_rng(seed)
    s = (rng.random(n) ** 3).astype(np.float32)
    if n >= 8:
        s[rng.integers(0, n, n // 8)] = np.float32(0.125)      # many equal scores
        s[rng.integers(0, n, n // 16)] = np.float32(0.0)
        s[rng.integers(0, n, 2)] = np.float32(np.inf)
    return s


@pytest.mark.parametrize("n", [1, 2, 255, 256, 257, 5000, 70001, 600000])
def test_topn_mask_bit_exact(n):
    import torch
    s = scores_with_ties(n, 3100 + n)
    sd = torch.from_numpy(s).cuda()
    cuts = sorted(set([0, n] + [int(x) for x in np.random.default_rng(n).integers(0, n + 1, 5)]))
    for N in sorted(set([0, 1, n // 3, n // 2, max(n - 1, 0), n])):
        if N > n:
            continue
        mask, counts = alcs.alcs_topn_mask(sd, N, seg_starts=cuts)
        want = oracle.topn_mask(s, N)
        got = mask.cpu().numpy()
        assert got.tobytes() == want.tobytes(), "n=%d N=%d" % (n, N)
        assert list(counts) == [int(want[a:b].sum()) for a, b in zip(cuts, cuts[1:])]
        _, c2 = alcs.alcs_topn_mask(sd, N, want_mask=False)
        assert list(c2) == [N]


def test_topn_with_nan_scores_ranks_them_above_infinity():
    import torch
    s = np.array([1.0, np.nan, np.inf, 0.5, np.nan, 3.0], dtype=np.float32)
    for N in range(7):
        mask, _ = alcs.alcs_topn_mask(torch.from_numpy(s).cuda(), N)
        assert mask.cpu().numpy().tobytes() == oracle.topn_mask(s, N).tobytes()
    mask, _ = alcs.alcs_topn_mask(torch.from_numpy(s).cuda(), 2)
    assert list(mask.cpu().numpy()) == [0, 1, 0, 0, 1, 0]


def test_topn_all_scores_equal_keeps_the_lowest_indices():
    import torch
    s = np.full(1000, 2.5, dtype=np.float32)
    mask, _ = alcs.alcs_topn_mask(torch.from_numpy(s).cuda(), 300)
    got = mask.cpu().numpy()
    assert got[:300].all() and not got[300:].any()


def synthetic_network(seed, scale=1):
    """Layer shapes of the MobileNetV1 pointwise convs (scaled down), Gaussian weights with a
    per-layer magnitude, and latency tables shaped like measured ones (a floor plus a slope)."""
    rng = np.random.default_rng(seed)
    shapes = [(32, 64), (64, 128), (128, 128), (128, 256), (256, 256), (256, 512)] + [(512, 512)] * 5 + \
             [(512, 1024), (1024, 1024)]
    Ws, tables = [], []
    for (ci, co) in shapes:
        ci, co = max(4, ci // scale), max(4, co // scale)
        Ws.append((rng.standard_normal((co, ci, 1, 1)) * (0.05 + rng.random() * 0.2)).astype(np.float32))
        nw = float(co * ci)
        k = np.arange(11) * 0.1 * nw
        floor, slope = 8.0 + 10 * rng.random(), (20 + 40 * rng.random()) / nw
        t = floor + slope * k * (1.0 + 0.1 * np.sin(np.arange(11)))      # locally linear, not globally
        tables.append((k, np.maximum.accumulate(t)))
    return Ws, tables


@pytest.mark.parametrize("seed,scale,frac", [(1, 8, 0.5), (2, 8, 0.2), (3, 4, 0.8), (4, 1, 0.45)])
def test_projection_matches_the_oracle(seed, scale, frac):
    import torch
    Ws, tables = synthetic_network(3200 + seed, scale)
    V = 4
    sc_dev = [alcs.alcs_block_scores(torch.from_numpy(W).cuda(), V) for W in Ws]
    sc_ref = [oracle.block_scores(W, V) for W in Ws]
    for a, b in zip(sc_dev, sc_ref):
        assert a.cpu().numpy().tobytes() == b.tobytes()
    starts = np.concatenate([[0], np.cumsum([s.size for s in sc_ref])]).astype(np.int64)
    allsc = torch.cat([s.reshape(-1) for s in sc_dev])
    tau = 25.0
    t_none = tau + sum(t[0] for _, t in tables)
    t_all = tau + sum(t[-1] for _, t in tables)
    budget = t_none + frac * (t_all - t_none)
    eps = 1e-3
    N, mask, t0, t1 = alcs.alcs_project_latency(allsc, starts, [V] * len(Ws), tables, tau, budget, eps)
    Nr, masks_r, t0r, t1r = oracle.project_latency(sc_ref, [V] * len(Ws), tables, tau, budget, eps)
    assert N == Nr
    assert abs(t0 - t0r) <= 1e-9 * t0r and abs(t1 - t1r) <= 1e-9 * t1r
    assert t0 < budget <= t1 or t1 - t0 <= eps
    want = np.concatenate([m.reshape(-1) for m in masks_r])
    assert mask.cpu().numpy().tobytes() == want.tobytes()
    # the projected network can be packed and its latency estimate honours the bracket
    nnz = [float(int(m.sum()) * V) for m in masks_r]
    assert t0 - 1e-9 <= alcs.alcs_network_latency(tau, tables, nnz) <= t1 + 1e-9


@pytest.mark.parametrize("layers,blocks,knots,kind", [(1, 1, 2, "rising"), (2, 300, 3, "rising"), (65, 40, 11, "ties"),
                                                      (5, 5000, 11, "equal"), (7, 900, 11, "falling"), (3, 700, 65, "rising"),
                                                      (1025, 3, 2, "rising")])
def test_projection_edges(layers, blocks, knots, kind):
    """Bisection on the device at its edges - one block, more layers than a wavefront, equal scores
    across layers, latency tables that do not rise - and the path beyond its layer and table limits."""
    import torch
    rng = np.random.default_rng(3400 + layers + blocks)
    sizes = rng.integers(1, blocks + 1, layers)
    sc = [(rng.random((int(m), 1, 1, 1)) ** 4 * (0.1 + rng.random())).astype(np.float32) for m in sizes]
    if kind == "ties":
        sc = [np.round(s * 20).astype(np.float32) for s in sc]
    if kind == "equal":
        sc = [np.full_like(s, 0.75) for s in sc]
    tables = []
    for m in sizes:
        k = np.arange(knots) * (4.0 * m / (knots - 1))
        t = 3.0 + 0.01 * k + 0.002 * m * rng.random(knots)
        tables.append((k, t if kind == "falling" else np.maximum.accumulate(t)))
    starts = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    allsc = torch.from_numpy(np.concatenate([s.reshape(-1) for s in sc])).cuda()
    t_none, t_all = sum(t[0] for _, t in tables), sum(t[-1] for _, t in tables)
    for frac, eps in ((0.0, 1e-3), (0.31, 1e-6), (0.7, 0.5), (2.0, 1e-3)):
        budget = t_none + frac * (t_all - t_none)
        N, mask, t0, t1 = alcs.alcs_project_latency(allsc, starts, [4] * layers, tables, 1.5, 1.5 + budget, eps)
        Nr, masks_r, t0r, t1r = oracle.project_latency(sc, [4] * layers, tables, 1.5, 1.5 + budget, eps)
        assert N == Nr, (frac, N, Nr)
        assert abs(t0 - t0r) <= 1e-9 * abs(t0r) and abs(t1 - t1r) <= 1e-9 * abs(t1r)
        assert mask.cpu().numpy().tobytes() == np.concatenate([m.reshape(-1) for m in masks_r]).tobytes(), frac


def bisect_on_host(scores, sizes, V, tables, tau, budget, eps):
    """Algorithm 1 with the library's own latency model, a comparison at a time; NaN is "not below"."""
    starts = np.concatenate([[0], np.cumsum(sizes)])

    def latency(N):
        m = oracle.topn_mask(scores, N)
        return alcs.alcs_network_latency(tau, tables, [float(V * int(m[a:b].sum())) for a, b in zip(starts, starts[1:])])

    N0, N1 = 0, int(scores.size)
    t0, t1 = latency(N0), latency(N1)
    while t1 - t0 > eps and N1 - N0 > 1:
        N = (N0 + N1) // 2
        t = latency(N)
        if t < budget:
            t0, N0 = t, N
        else:
            t1, N1 = t, N
    return (N0 + N1) // 2, oracle.topn_mask(scores, (N0 + N1) // 2), t0, t1


@pytest.mark.parametrize("times", [(0.0, -1e308, 1e308), (1.0, 1.7e308, 1.75e308), (-1.7e308, 0.5, 1.7e308), (0.0, 1e301, 2e301)])
@pytest.mark.parametrize("layers,blocks", [(1, 64), (3, 900)])
def test_projection_where_latencies_overflow(layers, blocks, times):
    """Finite tables whose neighbouring entries, or whose sums over the layers, a double does not hold:
    latencies are infinite or NaN, and the bisection ends as the comparisons say."""
    import torch
    rng = np.random.default_rng(3450 + layers)
    sizes = [blocks] * layers
    sc = (rng.random(blocks * layers) ** 3).astype(np.float32)
    tables = [(np.array([0.0, 2.0 * m, 4.0 * m]), np.array(times)) for m in sizes]
    starts = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    dev = torch.from_numpy(sc).cuda()
    for budget in (-1e307, 0.25, 1e300, float("inf"), -float("inf")):
        for eps in (1e-3, 1e305, float("inf")):
            N, mask, t0, t1 = alcs.alcs_project_latency(dev, starts, [4] * layers, tables, 1.5, budget, eps)
            Nr, mr, t0r, t1r = bisect_on_host(sc, sizes, 4, tables, 1.5, budget, eps)
            assert N == Nr, (budget, eps)
            assert np.array_equal([t0, t1], [t0r, t1r], equal_nan=True), (budget, eps)
            assert mask.cpu().numpy().tobytes() == mr.tobytes()


def test_projection_feeds_the_packer():
    """The mask that comes out of the projection is the mask alcs_pack_weights takes."""
    import torch
    rng = np.random.default_rng(3300)
    W = rng.standard_normal((64, 48, 1, 1)).astype(np.float32)
    sc = alcs.alcs_block_scores(torch.from_numpy(W).cuda(), 4)
    k = np.arange(11) * 0.1 * W.size
    N, mask, _, _ = alcs.alcs_project_latency(sc.reshape(-1), [0, sc.numel()], [4], [(k, 5.0 + 0.01 * k)], 0.0,
                                              5.0 + 0.01 * 0.3 * W.size, 1e-6)
    m = mask.cpu().numpy().reshape(16, 48, 1, 1)
    assert abs(int(m.sum()) - round(0.3 * 16 * 48)) <= 1
    packed = alcs.alcs_pack_weights(W, m, 4)
    assert packed.nnzb == int(m.sum())
    for got, want in zip(packed.export(), oracle.pack(W, m, 4)):
        assert got.tobytes() == want.tobytes()
    packed.free()


def test_rejected_arguments():
    import torch
    lib = alcs.load_library()
    s = torch.zeros(100, device="cuda")
    ws = torch.zeros(1024, dtype=torch.int64, device="cuda")
    P = lambda t: ctypes.c_void_p(t.data_ptr())
    LL = ctypes.c_longlong
    assert lib.alcs_topn_mask(P(s), LL(100), LL(101), None, 0, None, None, P(ws), None) < 0
    assert lib.alcs_topn_mask(P(s), LL(100), LL(-1), None, 0, None, None, P(ws), None) < 0
    assert lib.alcs_topn_mask(None, LL(100), LL(5), None, 0, None, None, P(ws), None) < 0
    assert lib.alcs_topn_mask(P(s), LL(100), LL(5), None, 0, None, None, None, None) < 0
    bad = (ctypes.c_longlong * 3)(0, 120, 100)
    assert lib.alcs_topn_mask(P(s), LL(100), LL(5), bad, 2, None, None, P(ws), None) < 0
    assert lib.alcs_block_scores(P(s), 4, 4, 1, 3, P(s), None) < 0          # V = 3
    assert lib.alcs_block_scores(P(s), 4, 4, 5, 4, P(s), None) < 0          # kernel = 5
    torch.cuda.synchronize()


@pytest.mark.parametrize("layers,knots", [(256, 6), (257, 5), (128, 12), (128, 13), (24, 64)])
def test_projection_at_the_limits_of_the_staged_tables(layers, knots):
    """256 layers and 1536 table entries are copied to LDS, more are read from memory: the same result."""
    import torch
    rng = np.random.default_rng(3500 + layers + knots)
    sizes = rng.integers(1, 60, layers)
    sc = [(rng.random((int(m), 1, 1, 1)) ** 3).astype(np.float32) for m in sizes]
    tables = [(np.arange(knots) * (4.0 * m / (knots - 1)), np.maximum.accumulate(2.0 + 0.02 * m * rng.random(knots))) for m in sizes]
    starts = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    none, every = sum(t[0] for _, t in tables), sum(t[-1] for _, t in tables)
    args = ([4] * layers, tables, 0.5, 0.5 + none + 0.4 * (every - none), 1e-4)
    N, mask, t0, t1 = alcs.alcs_project_latency(torch.from_numpy(np.concatenate([s.reshape(-1) for s in sc])).cuda(), starts, *args)
    Nr, masks_r, t0r, t1r = oracle.project_latency(sc, *args)
    assert N == Nr and abs(t0 - t0r) <= 1e-9 * t0r and abs(t1 - t1r) <= 1e-9 * t1r
    assert mask.cpu().numpy().tobytes() == np.concatenate([m.reshape(-1) for m in masks_r]).tobytes()
