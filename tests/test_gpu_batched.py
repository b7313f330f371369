"""GPU parity of the batched small-problem path (config 4: many graph-pair
sized problems with deletion rows/columns, Sec. 6) against the oracle, pair by
pair."""
import numpy as np
import pytest
import torch

import oracle
import workloads

pytestmark = pytest.mark.gpu


def _oracle_pair(B, p, mode, bp=True):
    Xp = B.X[B.x_off[p]:B.x_off[p + 1]]
    Yp = B.Y[B.y_off[p]:B.y_off[p + 1]]
    n, m = len(Xp), len(Yp)
    lam = float(B.lam[p])
    Bl = oracle.build_problem(Xp, Yp, B.cost, lam, mode, B.num_landmarks, B.landmark_seed + p, B.kmeans_iters,
                              B.ridge, 0, B.num_buckets, 1, B.lsh_seed + p)
    if bp:
        kpe = np.exp(-B.del_x[B.x_off[p]:B.x_off[p + 1]].astype(np.float64) / lam)
        keq = np.exp(-B.del_y[B.y_off[p]:B.y_off[p + 1]].astype(np.float64) / lam)
        a = np.full(n + m, 1.0 / (n + m))
        st = oracle.sinkhorn_bp(Bl.op, kpe, keq, a, a, B.iters)
        _, _, dist, resid = oracle.marginals_bp(Bl.op, kpe, keq, a, a, lam, st)
    else:
        a, b = np.full(n, 1.0 / n), np.full(m, 1.0 / m)
        st = oracle.sinkhorn(Bl.op, a, b, B.iters)
        _, _, dist, resid = oracle.marginals(Bl.op, a, b, lam, st)
    return Bl, st, dist, resid


def _run_gpu(B, mode, bp=True):
    import paper_2107_06876_amd as lcn
    dev = "cuda:0"
    modes = {"dense": lcn.MODE_DENSE, "sparse": lcn.MODE_SPARSE, "nystrom": lcn.MODE_NYSTROM, "lcn": lcn.MODE_LCN}
    X = torch.from_numpy(B.X).to(dev)
    Y = torch.from_numpy(B.Y).to(dev)
    dx = torch.from_numpy(B.del_x).to(dev) if bp else None
    dy = torch.from_numpy(B.del_y).to(dev) if bp else None
    lm = dict(num_landmarks=B.num_landmarks, kmeans_iters=B.kmeans_iters, seed=B.landmark_seed, ridge=B.ridge)
    lsh = dict(num_buckets=B.num_buckets, num_rounds=1, kmeans_iters=B.kmeans_iters, seed=B.lsh_seed)
    h = lcn.lcn_build_batched(X, Y, B.x_off, B.y_off, B.lam, B.cost, modes[mode], dx, dy,
                              landmarks=lm if mode in ("lcn", "nystrom") else None,
                              lsh=lsh if mode in ("lcn", "sparse") else None)
    status = lcn.sinkhorn_run(h, B.iters, check=False)
    dist, resid = lcn.lcn_batched_results(h)
    st = lcn.lcn_batched_get(h)
    st = {k: v.cpu().numpy() for k, v in st.items()}
    st["status"] = status
    st["counts"] = lcn.lcn_last_error_counts(h)
    return h, dist, resid, st


@pytest.mark.parametrize("mode,bp", [("lcn", True), ("dense", True), ("lcn", False), ("nystrom", True),
                                     ("sparse", True), ("sparse", False), ("dense", False)])
def test_config4(mode, bp):
    """All 1024 pairs of the configuration (Sec. 6 workload), every pair against the oracle's run of
    the same pair.  Without deletion entries the sparse kernel of a pair often has points whose
    bucket holds no point of the other set (4 buckets over 16..64 points): those get scaling 0 on
    both sides, are counted, and the call returns the warning status (App. "Limitations")."""
    import paper_2107_06876_amd as lcn
    B = workloads.config4()
    assert B.num_problems == 1024
    h, dist, resid, st = _run_gpu(B, mode, bp)
    worst = dict(log=0.0, cost=0.0, resid=0.0)
    counts_o = np.zeros(3, dtype=np.int64)
    for p in range(B.num_problems):
        Bl, so, dist_o, resid_o = _oracle_pair(B, p, mode, bp)
        n = int(B.x_off[p + 1] - B.x_off[p])
        m = int(B.y_off[p + 1] - B.y_off[p])
        z0 = int(B.x_off[p] + B.y_off[p])
        lu = st["log_u"][z0:z0 + (n + m if bp else n)]
        lv = st["log_v"][z0:z0 + (n + m if bp else m)]
        assert so.nonpositive == 0
        counts_o += (so.nonpositive, so.empty_rows, so.empty_cols)
        if mode in ("lcn", "nystrom"):
            np.testing.assert_array_equal(st["landmarks"][p], Bl.landmarks)
        if mode in ("lcn", "sparse"):
            np.testing.assert_array_equal(st["buckets"][z0:z0 + n + m], Bl.buckets[0])
        np.testing.assert_allclose(st["kernel"][p][:n, :m], Bl.op.dense(), rtol=2e-6, atol=1e-30)
        fu, fv = np.isfinite(so.log_u), np.isfinite(so.log_v)
        np.testing.assert_array_equal(np.isfinite(lu), fu)       # unsupported points: -infinity on both sides
        np.testing.assert_array_equal(np.isfinite(lv), fv)
        assert np.all(lu[~fu] == -np.inf) and np.all(lv[~fv] == -np.inf)
        worst["log"] = max(worst["log"], np.abs(lu - so.log_u)[fu].max(initial=0.0),
                           np.abs(lv - so.log_v)[fv].max(initial=0.0))
        worst["cost"] = max(worst["cost"], abs(dist[p] - dist_o) / abs(dist_o))
        worst["resid"] = max(worst["resid"], abs(resid[p] - resid_o))
    print("C4", mode, bp, worst, "status", st["status"], "counts", st["counts"], flush=True)
    assert worst["log"] <= 1e-4 and worst["cost"] <= 1e-4 and worst["resid"] <= 1e-5, worst
    assert st["counts"] == tuple(int(c) for c in counts_o)
    want = lcn.binding.WARN_NO_SUPPORT if counts_o[1] + counts_o[2] else lcn.binding.OK
    assert st["status"] == want
    if mode == "sparse" and not bp:
        assert counts_o[1] > 0 and counts_o[2] > 0    # the case this configuration exists to cover


def test_deletion_costs_bitwise():
    """c_i = || alpha .* x_i ||_2 (Sec. 6): same fp64 operations in the same order on both sides."""
    import paper_2107_06876_amd as lcn
    rng = np.random.default_rng(11)
    for total, d in ((1, 1), (257, 32), (5000, 64), (300, 301)):
        X = rng.standard_normal((total, d)).astype(np.float32)
        alpha = rng.uniform(0.5, 1.5, d).astype(np.float32)
        got = lcn.lcn_deletion_costs(torch.from_numpy(X).cuda(), torch.from_numpy(alpha).cuda()).cpu().numpy()
        np.testing.assert_array_equal(got, oracle.deletion_costs(X, alpha))
    empty = lcn.lcn_deletion_costs(torch.empty((0, 8), device="cuda"), torch.ones(8, device="cuda"))
    assert empty.numel() == 0


def test_multi_head_unbalanced():
    """Multi-head OT with learnable deletion costs (Sec. 6): every (pair, head) is a problem of
    the batch with lambda_k = 2^(k - K/2) lambda and c = || alpha_k .* x ||_2; the K distances
    of every pair against the oracle's."""
    import paper_2107_06876_amd as lcn
    H = workloads.config4_heads(pairs=40, heads=4)
    B, K = H.batch, H.heads
    P = B.num_problems
    dev = "cuda:0"
    X = torch.from_numpy(B.X).to(dev)
    Y = torch.from_numpy(B.Y).to(dev)
    lam = np.concatenate([lcn.lcn_head_lambdas(float(l0), K) for l0 in H.base_lam])
    dx = torch.empty(X.shape[0], dtype=torch.float32, device=dev)
    dy = torch.empty(Y.shape[0], dtype=torch.float32, device=dev)
    for q in range(P):                                    # one head's rows at a time
        a = torch.from_numpy(H.alpha[H.head_of[q]]).to(dev)
        lcn.lcn_deletion_costs(X[B.x_off[q]:B.x_off[q + 1]], a, out=dx[B.x_off[q]:B.x_off[q + 1]])
        lcn.lcn_deletion_costs(Y[B.y_off[q]:B.y_off[q + 1]], a, out=dy[B.y_off[q]:B.y_off[q + 1]])
    lm = dict(num_landmarks=B.num_landmarks, kmeans_iters=B.kmeans_iters, seed=B.landmark_seed, ridge=B.ridge)
    lsh = dict(num_buckets=B.num_buckets, num_rounds=1, kmeans_iters=B.kmeans_iters, seed=B.lsh_seed)
    h = lcn.lcn_build_batched(X, Y, B.x_off, B.y_off, lam, B.cost, lcn.MODE_LCN, dx, dy, landmarks=lm, lsh=lsh)
    lcn.sinkhorn_run(h, B.iters)
    dist, resid = lcn.lcn_batched_results(h)
    st = {k: v.cpu().numpy() for k, v in lcn.lcn_batched_get(h).items()}

    # the oracle's side: its own lambdas and deletion costs
    B.lam = np.concatenate([oracle.head_lambdas(float(l0), K) for l0 in H.base_lam])
    np.testing.assert_array_equal(lam, B.lam)
    B.del_x = np.concatenate([oracle.deletion_costs(B.X[B.x_off[q]:B.x_off[q + 1]], H.alpha[H.head_of[q]])
                              for q in range(P)])
    B.del_y = np.concatenate([oracle.deletion_costs(B.Y[B.y_off[q]:B.y_off[q + 1]], H.alpha[H.head_of[q]])
                              for q in range(P)])
    np.testing.assert_array_equal(dx.cpu().numpy(), B.del_x)
    np.testing.assert_array_equal(dy.cpu().numpy(), B.del_y)
    worst = dict(log=0.0, cost=0.0, resid=0.0)
    dist_o = np.empty(P)
    for q in range(P):
        Bl, so, dist_o[q], resid_o = _oracle_pair(B, q, "lcn", True)
        n = int(B.x_off[q + 1] - B.x_off[q])
        m = int(B.y_off[q + 1] - B.y_off[q])
        z0 = int(B.x_off[q] + B.y_off[q])
        assert so.nonpositive == 0
        np.testing.assert_array_equal(st["landmarks"][q], Bl.landmarks)
        np.testing.assert_array_equal(st["buckets"][z0:z0 + n + m], Bl.buckets[0])
        worst["log"] = max(worst["log"], np.abs(st["log_u"][z0:z0 + n + m] - so.log_u).max(),
                           np.abs(st["log_v"][z0:z0 + n + m] - so.log_v).max())
        worst["cost"] = max(worst["cost"], abs(dist[q] - dist_o[q]) / abs(dist_o[q]))
        worst["resid"] = max(worst["resid"], abs(resid[q] - resid_o))
    print("C4 heads", worst, flush=True)
    assert worst["log"] <= 1e-4 and worst["cost"] <= 1e-4 and worst["resid"] <= 1e-5, worst
    # d in R^K per pair: heads of a pair differ (their lambdas do)
    d_pk = dist.reshape(-1, K)
    assert np.all(np.ptp(d_pk, axis=1) > 0)


def test_batched_runs_resume():
    """sinkhorn_run(20) then sinkhorn_run(30) equals sinkhorn_run(50): the state between runs is
    the stored log scalings."""
    import paper_2107_06876_amd as lcn
    B = workloads.config4(pairs=64)
    dev = "cuda:0"
    X, Y = torch.from_numpy(B.X).to(dev), torch.from_numpy(B.Y).to(dev)
    dx, dy = torch.from_numpy(B.del_x).to(dev), torch.from_numpy(B.del_y).to(dev)
    lm = dict(num_landmarks=B.num_landmarks, kmeans_iters=B.kmeans_iters, seed=B.landmark_seed, ridge=B.ridge)
    lsh = dict(num_buckets=B.num_buckets, num_rounds=1, kmeans_iters=B.kmeans_iters, seed=B.lsh_seed)
    out = []
    for parts in ((50,), (20, 30)):
        h = lcn.lcn_build_batched(X, Y, B.x_off, B.y_off, B.lam, B.cost, lcn.MODE_LCN, dx, dy, landmarks=lm, lsh=lsh)
        for it in parts:
            lcn.sinkhorn_run(h, it)
        dist, resid = lcn.lcn_batched_results(h)
        dist2, _ = lcn.lcn_batched_results(h)                 # a query leaves the state alone
        np.testing.assert_array_equal(dist, dist2)
        st = lcn.lcn_batched_get(h)
        out.append((dist, st["log_u"].cpu().numpy(), st["log_v"].cpu().numpy()))
        lcn.lcn_destroy(h)
    np.testing.assert_allclose(out[0][0], out[1][0], rtol=1e-10)
    np.testing.assert_allclose(out[0][1], out[1][1], rtol=0, atol=1e-11)
    np.testing.assert_allclose(out[0][2], out[1][2], rtol=0, atol=1e-11)


def _edge_batch(sizes, d, l, b, rounds=1, seed=3):
    """A hand-made batch: sizes = [(n_p, m_p), ...]."""
    rng = np.random.default_rng(seed)
    ns = np.array([s[0] for s in sizes])
    ms = np.array([s[1] for s in sizes])
    x_off = np.concatenate([[0], np.cumsum(ns)]).astype(np.int64)
    y_off = np.concatenate([[0], np.cumsum(ms)]).astype(np.int64)
    X = rng.standard_normal((int(x_off[-1]), d)).astype(np.float32)
    Y = (rng.standard_normal((int(y_off[-1]), d)) + 0.2).astype(np.float32)
    lam = np.full(len(sizes), 0.5 * d, dtype=np.float32)
    B = workloads.Batch("edge", X, Y, x_off, y_off, lam,
                        rng.uniform(0.5, 2.0, X.shape[0]).astype(np.float32),
                        rng.uniform(0.5, 2.0, Y.shape[0]).astype(np.float32),
                        workloads.COST_EUCLID, num_landmarks=l, num_buckets=b, iters=30)
    return B


@pytest.mark.parametrize("d,l,b", [(1, 1, 1), (64, 2, 2), (7, 2, 1)])
@pytest.mark.parametrize("mode,bp", [("lcn", True), ("lcn", False), ("sparse", True), ("dense", False)])
def test_batched_edge_shapes(d, l, b, mode, bp):
    """Pairs of 1 x 1, 64 x 64 (the largest), 1 x 64 and 64 x 1 points and ragged ones in one batch;
    one dimension and 64; one landmark, one bucket; per-point deletion costs."""
    sizes = [(1, 1), (64, 64), (1, 64), (64, 1), (17, 33), (2, 2), (63, 64)]
    B = _edge_batch(sizes, d, l, b)
    h, dist, resid, st = _run_gpu(B, mode, bp)
    worst = dict(log=0.0, cost=0.0, resid=0.0)
    for p in range(B.num_problems):
        Bl, so, dist_o, resid_o = _oracle_pair(B, p, mode, bp)
        n, m = sizes[p]
        z0 = int(B.x_off[p] + B.y_off[p])
        if so.nonpositive:
            continue   # the Nystrom part went negative on this pair: the batch reports it (checked below)
        lu = st["log_u"][z0:z0 + (n + m if bp else n)]
        lv = st["log_v"][z0:z0 + (n + m if bp else m)]
        if mode == "lcn":
            np.testing.assert_array_equal(st["landmarks"][p], Bl.landmarks)
        if mode in ("lcn", "sparse"):
            np.testing.assert_array_equal(st["buckets"][z0:z0 + n + m], Bl.buckets[0])
        fin = np.isfinite(so.log_u)
        worst["log"] = max(worst["log"], np.abs(lu - so.log_u)[fin].max(initial=0.0),
                           np.abs(lv - so.log_v)[np.isfinite(so.log_v)].max(initial=0.0))
        worst["cost"] = max(worst["cost"], abs(dist[p] - dist_o) / abs(dist_o))
        worst["resid"] = max(worst["resid"], abs(resid[p] - resid_o))
    print("C4 edge", d, l, b, mode, bp, worst, flush=True)
    assert worst["log"] <= 1e-4 and worst["cost"] <= 1e-4 and worst["resid"] <= 1e-5, worst


@pytest.mark.parametrize("mode,bp,lam", [("lcn", True, 4.0), ("dense", True, 0.12), ("dense", False, 0.12), ("sparse", True, 0.5)])
def test_batched_iteration_on_block_edges(mode, bp, lam):
    """The iteration deals a pair's kernel to the lanes in 8 x 8 blocks: sizes on both sides of a block,
    of a lane row and of the half-wavefront.  The small lambdas take the scalings far out of
    2^-40 .. 2^40, where the common exponent is taken out again."""
    sizes = [(8, 9), (7, 64), (33, 31), (16, 8), (24, 25), (1, 9), (64, 57), (15, 41)]
    d = 9
    B = _edge_batch(sizes, d, 2, 2, seed=11)
    B.lam[:] = lam
    # kernel entries are single precision: above e^-87 they are normal numbers and keep their 24 bits
    far = np.linalg.norm(B.X[:, None, :].astype(np.float64) - B.Y[None, :, :], axis=2).max()
    assert mode == "lcn" or far / lam < 87.0
    h, dist, resid, st = _run_gpu(B, mode, bp)
    for p, (n, m) in enumerate(sizes):
        Bl, so, dist_o, resid_o = _oracle_pair(B, p, mode, bp)
        assert so.nonpositive == 0
        z0 = int(B.x_off[p] + B.y_off[p])
        lu = st["log_u"][z0:z0 + (n + m if bp else n)]
        lv = st["log_v"][z0:z0 + (n + m if bp else m)]
        # the pair's kernel is stored in single precision: 2^-24 per entry and half-iteration at most adds up
        # over the 30 iterations (and is contracted by them), far below the parity bound
        np.testing.assert_allclose(lu, so.log_u, rtol=0, atol=1e-4)
        np.testing.assert_allclose(lv, so.log_v, rtol=0, atol=1e-4)
        assert abs(dist[p] - dist_o) <= 1e-4 * abs(dist_o) and abs(resid[p] - resid_o) <= 1e-5


@pytest.mark.parametrize("d,l,b,rounds,kind", [(16, 5, 3, 2, "plain"), (17, 16, 16, 4, "plain"), (33, 3, 4, 1, "ties"),
                                               (3, 9, 7, 3, "ties"), (8, 4, 4, 1, "large")])
def test_batched_build_decides_like_the_rule(d, l, b, rounds, kind):
    """Buckets and landmarks bit for bit: centroids of several k-means runs over one and several tiles of
    sixteen; points on a coarse grid, where many distances are exactly equal and the matrix product leaves
    every decision to the rule; coordinates above 2^13, where the member sums are integers."""
    sizes = [(16, 16), (17, 20), (64, 64), (33, 31), (40, 9)]
    B = _edge_batch(sizes, d, l, b, seed=7)
    if kind == "ties":
        B.X[:] = np.round(B.X)
        B.Y[:] = np.round(B.Y)
    if kind == "large":
        B.X *= 6000.0
        B.Y *= 6000.0
        B.lam[:] *= 6000.0
    import paper_2107_06876_amd as lcn
    import oracle
    dev = "cuda:0"
    lm = dict(num_landmarks=l, kmeans_iters=7, seed=3, ridge=0.5)
    lsh = dict(num_buckets=b, num_rounds=rounds, kmeans_iters=9, seed=41)
    h = lcn.lcn_build_batched(torch.from_numpy(B.X).to(dev), torch.from_numpy(B.Y).to(dev), B.x_off, B.y_off, B.lam,
                              B.cost, lcn.MODE_LCN, None, None, landmarks=lm, lsh=lsh)
    st = lcn.lcn_batched_get(h)
    landmarks, buckets = st["landmarks"].cpu().numpy(), st["buckets"].cpu().numpy()
    for p, (n, m) in enumerate(sizes):
        Z = np.concatenate([B.X[B.x_off[p]:B.x_off[p + 1]], B.Y[B.y_off[p]:B.y_off[p + 1]]])
        cent, _ = oracle.kmeans(Z, l, 7, 3 + p)
        np.testing.assert_array_equal(landmarks[p], cent)
        z0 = int(B.x_off[p] + B.y_off[p]) * rounds
        for r in range(rounds):
            _, asg = oracle.kmeans(Z, b, 9, 41 + p * rounds + r)
            np.testing.assert_array_equal(buckets[z0 + r * (n + m):z0 + (r + 1) * (n + m)], asg)
    lcn.lcn_destroy(h)


def _build_only(B, mode, lm, lsh):
    import paper_2107_06876_amd as lcn
    modes = {"dense": lcn.MODE_DENSE, "sparse": lcn.MODE_SPARSE, "nystrom": lcn.MODE_NYSTROM, "lcn": lcn.MODE_LCN}
    return lcn.lcn_build_batched(torch.from_numpy(B.X).cuda(), torch.from_numpy(B.Y).cuda(), B.x_off, B.y_off, B.lam,
                                 B.cost, modes[mode], None, None, landmarks=lm if mode in ("lcn", "nystrom") else None,
                                 lsh=lsh if mode in ("lcn", "sparse") else None)


@pytest.mark.parametrize("mode", ["sparse", "lcn"])
@pytest.mark.parametrize("what", [np.nan, np.inf])
def test_batched_points_that_are_not_finite(mode, what):
    """No distance of such a point is a finite number: it is in bucket 0 of every round, as the rule has it (the
    lowest index among equals; a first distance that is not a number is never beaten), the pair fails where its
    kernel has such entries, and the other pairs do not change by a bit."""
    import paper_2107_06876_amd as lcn
    sizes = [(20, 30), (33, 31), (16, 16), (64, 60)]
    d, l, b, rounds = 18, 5, 4, 2
    lm = dict(num_landmarks=l, kmeans_iters=6, seed=3, ridge=0.5)
    lsh = dict(num_buckets=b, num_rounds=rounds, kmeans_iters=6, seed=41)
    out = []
    for spoilt in (False, True):
        B = _edge_batch(sizes, d, l, b, seed=7)
        if spoilt:
            B.X[B.x_off[1] + 4, 3] = what
            B.Y[B.y_off[1] + 30, 17] = what
        h = _build_only(B, mode, lm, lsh)
        status = lcn.sinkhorn_run(h, 5, check=False)
        st = {k: v.cpu().numpy() for k, v in lcn.lcn_batched_get(h).items()}
        out.append((status, st))
        lcn.lcn_destroy(h)
    (_, clean), (status, st) = out
    if np.isnan(what):
        assert status == lcn.binding.ERR_NONPOSITIVE
    for p, (n, m) in enumerate(sizes):
        z0, N = int(B.x_off[p] + B.y_off[p]), n + m
        buckets = st["buckets"][z0 * rounds:(z0 + N) * rounds].reshape(rounds, N)
        if p == 1:
            assert buckets.min() >= 0 and buckets.max() < b
            assert (buckets[:, 4] == 0).all() and (buckets[:, n + 30] == 0).all()
            continue
        np.testing.assert_array_equal(buckets, clean["buckets"][z0 * rounds:(z0 + N) * rounds].reshape(rounds, N))
        np.testing.assert_array_equal(st["kernel"][p][:n, :m], clean["kernel"][p][:n, :m])
        np.testing.assert_array_equal(st["log_u"][z0:z0 + n], clean["log_u"][z0:z0 + n])
        np.testing.assert_array_equal(st["log_v"][z0:z0 + m], clean["log_v"][z0:z0 + m])
        if mode == "lcn":
            np.testing.assert_array_equal(st["landmarks"][p], clean["landmarks"][p])


@pytest.mark.parametrize("scale", [3e7, 1e8])
def test_batched_build_on_far_points(scale):
    """Coordinates above 2^24, where the 64-bit sum of 128 of them might wrap: the rule decides on every centroid."""
    import paper_2107_06876_amd as lcn
    sizes = [(16, 16), (17, 20), (40, 9)]
    B = _edge_batch(sizes, 8, 3, 4, seed=7)
    B.X *= scale / 4
    B.Y *= scale / 4
    B.lam[:] *= scale
    h = _build_only(B, "lcn", dict(num_landmarks=3, kmeans_iters=7, seed=3, ridge=0.5),
                    dict(num_buckets=4, num_rounds=2, kmeans_iters=9, seed=41))
    st = {k: v.cpu().numpy() for k, v in lcn.lcn_batched_get(h).items()}
    for p, (n, m) in enumerate(sizes):
        Z = np.concatenate([B.X[B.x_off[p]:B.x_off[p + 1]], B.Y[B.y_off[p]:B.y_off[p + 1]]])
        assert np.abs(Z.astype(np.float64).sum(axis=0)).max() * 2.0 ** 32 < 2.0 ** 63   # no sum wraps
        np.testing.assert_array_equal(st["landmarks"][p], oracle.kmeans(Z, 3, 7, 3 + p)[0])
        z0 = int(B.x_off[p] + B.y_off[p]) * 2
        for r in range(2):
            np.testing.assert_array_equal(st["buckets"][z0 + r * (n + m):z0 + (r + 1) * (n + m)],
                                          oracle.kmeans(Z, 4, 9, 41 + p * 2 + r)[1])


def _nystrom_extended(Z, n, L, lam, ridge, euclid):
    """U A^{-1} V of a pair in extended precision, and what double precision may change in it, to first order: an
    exponent from d differences is off by d + 2 roundings of itself and the exponential by two more; the solve by
    2 l roundings of the (unit) diagonal."""
    Z, L, lam = Z.astype(np.longdouble), L.astype(np.longdouble), np.longdouble(lam)

    def exponents(a, b):
        sq = ((a[:, None] - b[None]) ** 2).sum(-1)
        return (np.sqrt(sq) if euclid else sq) / lam
    (d, l), eF, eA = (Z.shape[1], len(L)), exponents(Z, L), exponents(L, L)
    F, A = np.exp(-eF), np.exp(-eA) + np.longdouble(ridge) * np.eye(l, dtype=np.longdouble)
    C, W, S = np.zeros_like(A), np.zeros_like(F), np.zeros_like(F)
    for j in range(l):
        C[j, j] = np.sqrt(A[j, j] - (C[j, :j] ** 2).sum())
        for i in range(j + 1, l):
            C[i, j] = (A[i, j] - (C[i, :j] * C[j, :j]).sum()) / C[j, j]
        W[:, j] = (F[:, j] - W[:, :j] @ C[j, :j]) / C[j, j]
    for j in reversed(range(l)):
        S[:, j] = (W[:, j] - S[:, j + 1:] @ C[j + 1:, j]) / C[j, j]
    S = np.abs(S)   # |F A^{-1}|
    dF, dA = ((d + 2) * eF + 2) * F, ((d + 2) * eA + 2) * A + 2 * l
    return W[:n] @ W[n:].T, 2.0 ** -53 * (dF[:n] @ S[n:].T + S[:n] @ dF[n:].T + S[:n] @ dA @ S[n:].T)


@pytest.mark.parametrize("cost,d,l,lam", [(workloads.COST_SQEUCLID, 2, 16, 2.0), (workloads.COST_SQEUCLID, 2, 16, 1.0),
                                          (workloads.COST_SQEUCLID, 5, 12, 0.6), (workloads.COST_EUCLID, 17, 9, 4.0)])
def test_batched_landmark_costs_away_from_the_origin(cost, d, l, lam):
    """Points whose norms are large against their distances: a cost from dot products would lose the digits that the
    norms have in common, and the inverse of the landmarks' matrix multiplies what is lost."""
    import paper_2107_06876_amd as lcn
    sizes = [(40, 50)] * 48
    B = _edge_batch(sizes, d, l, 2, seed=9)
    B.X[:, 0] += 70.0 * d ** 0.5
    B.Y[:, 0] += 70.0 * d ** 0.5
    B.cost = cost
    B.lam[:] = lam
    h = _build_only(B, "nystrom", dict(num_landmarks=l, kmeans_iters=1, seed=3, ridge=1e-10), None)
    st = {k: v.cpu().numpy() for k, v in lcn.lcn_batched_get(h).items()}
    lcn.lcn_destroy(h)
    worst = 0.0
    for p, (n, m) in enumerate(sizes):
        Z = np.concatenate([B.X[B.x_off[p]:B.x_off[p + 1]], B.Y[B.y_off[p]:B.y_off[p + 1]]])
        want, bound = _nystrom_extended(Z, n, st["landmarks"][p], B.lam[p], 1e-10, cost == workloads.COST_EUCLID)
        bound += 2.0 ** -24 * (np.abs(want) + bound)   # the entry is stored in single precision
        worst = max(worst, float((np.abs(st["kernel"][p][:n, :m] - want) / bound).max()))
    print("landmark costs", cost, d, l, lam, "largest error over its bound", worst, flush=True)
    assert worst <= 1.0


@pytest.mark.parametrize("d,l,b,rounds,kind,many", [(8, 5, 3, 2, "plain", True), (16, 16, 16, 4, "ties", True),
                                                    (12, 9, 7, 3, "large", True), (24, 9, 7, 3, "ties", True),
                                                    (32, 16, 16, 4, "plain", True), (20, 4, 4, 1, "large", True),
                                                    (17, 3, 16, 2, "large", True), (9, 7, 5, 3, "ties", False),
                                                    (31, 16, 9, 2, "plain", False), (50, 6, 6, 2, "ties", False)])
def test_batched_build_by_four_wavefronts(d, l, b, rounds, kind, many):
    """As above where four wavefronts build a pair: more than two pairs per compute unit (so that each holds two tiles of
    points; for up to 16 dimensions, up to 32, and one to five tiles of centroids, whose sums are split into parts or
    not), or pairs of at most 64 points; and eight wavefronts for more than 32 dimensions."""
    import paper_2107_06876_amd as lcn
    base = [(16, 16), (17, 20), (64, 64), (33, 31), (40, 9)] if many else [(16, 16), (17, 20), (33, 31), (40, 9)]
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    sizes = base * ((2 * cus) // len(base) + 1) if many else base
    B = _edge_batch(sizes, d, l, b, seed=7)
    if kind == "ties":
        B.X[:] = np.round(B.X)
        B.Y[:] = np.round(B.Y)
    if kind == "large":
        B.X *= 6000.0
        B.Y *= 6000.0
        B.lam[:] *= 6000.0
    h = _build_only(B, "lcn", dict(num_landmarks=l, kmeans_iters=7, seed=3, ridge=0.5),
                    dict(num_buckets=b, num_rounds=rounds, kmeans_iters=9, seed=41))
    st = {k: v.cpu().numpy() for k, v in lcn.lcn_batched_get(h).items()}
    lcn.lcn_destroy(h)
    for p in sorted({*range(len(base)), *range(len(sizes) - len(base), len(sizes))}):
        n, m = sizes[p]
        Z = np.concatenate([B.X[B.x_off[p]:B.x_off[p + 1]], B.Y[B.y_off[p]:B.y_off[p + 1]]])
        np.testing.assert_array_equal(st["landmarks"][p], oracle.kmeans(Z, l, 7, 3 + p)[0])
        z0 = int(B.x_off[p] + B.y_off[p]) * rounds
        for r in range(rounds):
            np.testing.assert_array_equal(st["buckets"][z0 + r * (n + m):z0 + (r + 1) * (n + m)],
                                          oracle.kmeans(Z, b, 9, 41 + p * rounds + r)[1])


@pytest.mark.parametrize("many", [False, True])
@pytest.mark.parametrize("d,scale,offset", [(32, 1.0, 300.0), (16, 1.0, 1e6), (64, 2.0, -8000.0), (20, 3e-13, 0.0),
                                            (32, 1e-11, 0.0), (9, 0.0, 7.0), (31, 4000.0, 0.0)])
def test_batched_build_decides_like_the_rule_anywhere(d, scale, offset, many):
    """Scores in single precision about the middle of the points, member sums digit by digit: pairs far from the origin, squares
    near single precision's smallest numbers, points that all coincide, coordinates just below 2^13; the buckets
    are the rule's, bit for bit."""
    import paper_2107_06876_amd as lcn
    base = [(16, 16), (17, 20), (64, 64), (33, 31), (40, 9), (5, 4)]
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    sizes = base * ((2 * cus) // len(base) + 1) if many else base
    B = _edge_batch(sizes, d, 6, 5, seed=11)
    for Z in (B.X, B.Y):
        Z[:] = np.clip(Z * np.float32(scale), -8191.5, 8191.5) + np.float32(offset)
    B.lam[:] = 1.0
    h = _build_only(B, "sparse", None, dict(num_buckets=5, num_rounds=2, kmeans_iters=9, seed=41))
    st = {k: v.cpu().numpy() for k, v in lcn.lcn_batched_get(h).items()}
    for p in range(len(base)):
        n, m = sizes[p]
        Z = np.concatenate([B.X[B.x_off[p]:B.x_off[p + 1]], B.Y[B.y_off[p]:B.y_off[p + 1]]])
        z0 = int(B.x_off[p] + B.y_off[p]) * 2
        for r in range(2):
            np.testing.assert_array_equal(st["buckets"][z0 + r * (n + m):z0 + (r + 1) * (n + m)],
                                          oracle.kmeans(Z, 5, 9, 41 + p * 2 + r)[1])


@pytest.mark.parametrize("d,values,base,spread", [(8, 2, 2.0 ** -33, 0.7 * 2.0 ** -41), (32, 2, 2.0 ** -33, 0.7 * 2.0 ** -37),
                                                  (8, 3, 2.0 ** -33, 0.7 * 2.0 ** -37), (16, 3, 1.5 * 2.0 ** -32, 0.7 * 2.0 ** -40),
                                                  (48, 3, 2.0 ** -33, 0.7 * 2.0 ** -41)])
def test_batched_build_of_points_closer_than_a_means_rounding(d, values, base, spread):
    """Coordinates on either side of a tie of the 2^-32 fixed point that means are formed in, far closer together than
    that: the centroids leave the points' hull by many times its width.  600 pairs (a share of
    the first four cases' decided wrongly where the scores' bound took the centroids to be inside)."""
    import paper_2107_06876_amd as lcn
    sizes = [(16, 16), (9, 11), (20, 12), (13, 31), (10, 9), (8, 8), (64, 64), (40, 41)] * 75
    B = _edge_batch(sizes, d, 6, 16, seed=11)
    rng = np.random.default_rng(5)
    for Z in (B.X, B.Y):
        s = rng.integers(0, 2, Z.shape) * 2 - 1 if values == 2 else rng.integers(-1, 2, Z.shape)
        Z[:] = (base + spread * s).astype(np.float32)
    B.lam[:] = 1.0
    h = _build_only(B, "sparse", None, dict(num_buckets=16, num_rounds=1, kmeans_iters=9, seed=41))
    st = {k: v.cpu().numpy() for k, v in lcn.lcn_batched_get(h).items()}
    wrong = []
    for p, (n, m) in enumerate(sizes):
        Z = np.concatenate([B.X[B.x_off[p]:B.x_off[p + 1]], B.Y[B.y_off[p]:B.y_off[p + 1]]])
        z0 = int(B.x_off[p] + B.y_off[p])
        if not np.array_equal(st["buckets"][z0:z0 + n + m], oracle.kmeans(Z, 16, 9, 41 + p)[1]):
            wrong.append(p)
    assert wrong == []


def test_runs_of_two_batches_share_the_chip():
    """Four pairs per compute unit leave room for a second run on another stream.  Some 3 ms each: both together take 1.6
    times one (2.0 where the second has to wait for the first, also for want of a hardware queue of its own: the best of
    the pairs that four streams make counts)."""
    import itertools
    import threading
    import time
    import paper_2107_06876_amd as lcn
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    B = _edge_batch([(40, 41)] * (4 * cus), 8, 3, 4)
    X, Y, dx, dy = (torch.from_numpy(v).cuda() for v in (B.X, B.Y, B.del_x, B.del_y))
    torch.cuda.synchronize()
    handles = []
    for stream in [torch.cuda.Stream() for _ in range(4)]:
        with torch.cuda.stream(stream):
            handles.append(lcn.lcn_build_batched(X, Y, B.x_off, B.y_off, B.lam, B.cost, lcn.MODE_DENSE, dx, dy))

    def seconds(used):
        threads = [threading.Thread(target=lcn.sinkhorn_run, args=(h, 4000)) for h in used]
        start = time.perf_counter()
        for t in threads:
            t.start()
        for t in threads:
            t.join()
        return time.perf_counter() - start

    seconds(handles)
    one = min(seconds(handles[:1]) for _ in range(5))
    two = min(seconds(pair) for pair in itertools.combinations(handles, 2) for _ in range(3))
    print("one run %.2f ms, two runs %.2f ms" % (1e3 * one, 1e3 * two), flush=True)
    assert two < 1.8 * one


@pytest.mark.parametrize("pairs", [5, 256, 257, 258, 1023])
@pytest.mark.parametrize("bp", [True, False])
def test_marginals_left_by_a_run_or_formed_when_asked_for(pairs, bp):
    """A run leaves the marginals where the workspace has room for them; without it they are formed from the state, and so they are before
    any run.  Both are roundings of the same double precision sums (relative difference some 1e-15 before it).  Entries
    between the pairs are not written without deletion entries.  Up to a pair per compute unit (256) and more, the last
    workgroup of the run with one to three pairs."""
    import ctypes
    import paper_2107_06876_amd as lcn
    B = _edge_batch([(16 + (7 * p) % 49, 16 + (11 * p) % 49) for p in range(pairs)], 8, 3, 4)
    lsh = dict(num_buckets=4, num_rounds=1, kmeans_iters=3, seed=41)
    X, Y = torch.from_numpy(B.X).cuda(), torch.from_numpy(B.Y).cuda()
    dx = torch.from_numpy(B.del_x).cuda() if bp else None
    dy = torch.from_numpy(B.del_y).cuda() if bp else None
    total = len(B.X) + len(B.Y)

    def build(workspace):
        return lcn.lcn_build_batched(X, Y, B.x_off, B.y_off, B.lam, B.cost, lcn.MODE_DENSE, dx, dy, lsh=lsh, workspace=workspace)

    def results(h):
        dist, resid = np.empty(pairs), np.empty(pairs)
        rows, cols = torch.full((total,), -7.0, device="cuda"), torch.full((total,), -7.0, device="cuda")
        st = lcn.load_library().lcn_batched_results(h.raw, dist.ctypes.data, resid.ctypes.data, ctypes.c_void_p(rows.data_ptr()),
                                                    ctypes.c_void_p(cols.data_ptr()))
        assert st == 0
        return dist, resid, rows.cpu().numpy(), cols.cpu().numpy()

    need = build(torch.empty(256, dtype=torch.uint8, device="cuda")).workspace.numel()   # too little: built again with what is asked for
    room = build(torch.empty(need, dtype=torch.uint8, device="cuda"))
    none = build(torch.empty(need - 256 - 8 * total, dtype=torch.uint8, device="cuda"))   # taken, but the marginals do not fit
    assert need > 256 + 8 * total and none.workspace.numel() == need - 256 - 8 * total
    for iters in (0, 3, 2):
        if iters:
            lcn.sinkhorn_run(room, iters)
            lcn.sinkhorn_run(none, iters)
        got, want = results(room), results(none)
        np.testing.assert_allclose(got[0], want[0], rtol=1e-12, atol=1e-13)
        np.testing.assert_allclose(got[1], want[1], rtol=0, atol=1e-13)
        for g, w in zip(got[2:], want[2:]):
            np.testing.assert_array_equal(g == -7.0, w == -7.0)
            np.testing.assert_allclose(g, w, rtol=1.2e-7, atol=0)   # a rounding to single precision
