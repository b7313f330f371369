"""Sizes at which a kernel or a rule of a dispatch changes: rows per wavefront of a sweep, lanes per row of a sweep in logs,
ranges of points and clusters times points in the k-means update, pieces of the sparse values' tiles, pinned blocks
of batches.  Against the oracle (tolerances of parity.py), or against the exact rule applied to every point."""
import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu


def _cut(n, m, d, landmarks, buckets, rounds, iters, kmeans_iters=2, seed=11):
    """Unit-free points of two overlapping clouds, smooth enough for every sum to stay positive."""
    p = workloads.config3(n=64, d=8, landmarks=8, buckets=8, rounds=rounds, iters=iters, name="cut")
    rng = np.random.default_rng(seed)
    p.X = rng.standard_normal((n, d)).astype(np.float32)
    p.Y = (0.9 * rng.standard_normal((m, d)) + 0.1).astype(np.float32)
    p.a = (rng.random(n) + 0.5).astype(np.float32)
    p.b = (rng.random(m) + 0.5).astype(np.float32)
    p.a /= p.a.sum()
    p.b /= p.b.sum()
    p.cost, p.lam = workloads.COST_SQEUCLID, 4.0 * d
    p.num_landmarks, p.num_buckets, p.num_rounds, p.kmeans_iters = landmarks, buckets, rounds, kmeans_iters
    p.iters, p.ridge = iters, 1e-6
    return p


# a chip of 256 compute units has 4096 wavefronts: one, two, three and five rows per wavefront, then whichever of three and five
# takes fewer turns; short records (one wavefront of entries requested with a row of five) and long ones (two)
@pytest.mark.parametrize("n,m,landmarks,buckets,rounds", [
    (1, 4097, 20, 1, 1),          # a single row against thousands
    (4096, 4097, 20, 300, 1),     # one row per wavefront / two, up to 64 columns
    (8192, 8193, 70, 500, 2),     # two / three, up to 128 columns
    (12288, 12289, 140, 900, 3),  # three / five, up to 192 columns
    (20480, 20481, 30, 1500, 1),  # five / three, short records
    (24577, 12300, 20, 400, 2),   # three, unequal sides
    (13000, 12999, 40, 120, 1),   # five, long records
    (5000, 5001, 300, 200, 1),    # more than 256 columns
    (5000, 5001, 300, 20, 2),     # the same with long records: three wavefronts of entries requested with a row
])
def test_rows_per_wavefront(n, m, landmarks, buckets, rounds):
    from parity import compare
    print("rows", n, m, compare(_cut(n, m, 3, landmarks, buckets, rounds, 6), "lcn"), flush=True)


@pytest.mark.parametrize("groups", [63, 64, 65])
def test_totals_taken_directly_or_handed_over(monkeypatch, groups):
    """Up to 64 partial sums of 64 columns every workgroup adds up by itself, above that they are handed over; both give
    the bits of the separate reduction."""
    import torch
    import paper_2107_06876_amd as lcn
    from parity import gpu_build
    p = _cut(16 * groups, 16 * groups - 3, 4, 24, 40, 1, 8)
    got = {}
    for fused in ("1", "0"):
        monkeypatch.setenv("LCN_FUSED_REDUCE", fused)
        h = gpu_build(p, "lcn")
        lcn.sinkhorn_run(h, 5)
        lcn.sinkhorn_run(h, 3)
        got[fused] = lcn.lcn_get_scalings(h) + (lcn.transport_cost(h),)
        lcn.lcn_destroy(h)
    assert torch.equal(got["1"][0], got["0"][0]) and torch.equal(got["1"][1], got["0"][1])
    assert got["1"][2] == got["0"][2]


# records of a few entries up to hundreds, on both sides of the change from 16 to 32 lanes per row (40 entries of two to four
# rounds, 48 of more); 3001 and 9 rows: a last workgroup partly empty; five rounds: unrolled over eight
@pytest.mark.parametrize("n,m,buckets,rounds", [(3001, 2999, 700, 1), (3001, 2999, 60, 1), (2000, 2001, 150, 2),
                                               (1500, 1499, 40, 3), (1200, 1201, 60, 4), (1000, 999, 60, 5), (9, 700, 3, 1)])
def test_lanes_per_row_in_logs(n, m, buckets, rounds):
    from parity import compare
    print("logs", n, m, buckets, rounds, compare(_cut(n, m, 4, 8, buckets, rounds, 12), "sparse"), flush=True)


# records of several rounds: short pieces (up to 28 entries on average) and longer ones, fewer than 8000 and 12 000 rows and more,
# one round of long pieces; empty rounds of a row
@pytest.mark.parametrize("n,m,buckets,rounds", [(12100, 11900, 560, 2), (7000, 6900, 70, 2), (7999, 8001, 100, 3), (12001, 11999, 300, 4),
                                               (12500, 12100, 80, 3), (12500, 12100, 80, 2), (6100, 6000, 13, 1), (3000, 40, 30, 3)])
def test_rounds_of_a_record_in_logs(n, m, buckets, rounds):
    from parity import compare
    print("logs", n, m, buckets, rounds, compare(_cut(n, m, 4, 8, buckets, rounds, 3), "sparse"), flush=True)


# each choice of log_walk.h for two to four rounds, the lines between them lying between the two sides' numbers of rows
@pytest.mark.parametrize("n,m,buckets,rounds", [(10003, 9997, 190, 3), (5003, 4997, 300, 3), (5001, 4996, 240, 2), (7999, 8001, 40, 2),
                                               (12001, 11999, 40, 2), (18001, 17999, 70, 3), (3000, 12001, 14, 3), (12003, 11997, 1000, 4)])
def test_walks_of_a_record_in_logs(n, m, buckets, rounds):
    from parity import compare
    print("walks", n, m, buckets, rounds, compare(_cut(n, m, 4, 8, buckets, rounds, 3), "sparse"), flush=True)


# the bucket sort: buckets on both sides of 256 (a wavefront's share of a scan) and of a power of two (bits of a key), blocks on both
# sides of 1024 (a workgroup's), points on both sides of 1024 (a chunk), eight chunks and more, of 4096 (rows of a scan's tile)
@pytest.mark.parametrize("n,m,buckets,rounds", [(1024, 1025, 256, 1), (8193, 7, 257, 2), (3000, 4097, 342, 3), (4096, 2000, 1025, 1),
                                               (9000, 8191, 512, 2), (600, 601, 130, 8)])
def test_bucket_sort_edges(n, m, buckets, rounds):
    from parity import compare
    print("sort", n, m, buckets, rounds, compare(_cut(n, m, 3, 8, buckets, rounds, 2), "sparse"), flush=True)


# more than four rounds: their words are looked up as the walk reaches them; several rounds ending in one piece of 64
# entries, empty ones, ones longer than a trip; every width of the sweeps and rows per wavefront
@pytest.mark.parametrize("n,m,landmarks,buckets,rounds", [
    (300, 301, 20, 40, 5), (40, 41, 8, 80, 8), (2500, 2501, 20, 4, 6), (4100, 4099, 70, 60, 7), (9000, 8999, 140, 100, 5),
    (17000, 17001, 130, 2600, 8), (17000, 16999, 250, 300, 6), (2000, 1999, 300, 30, 5), (1500, 1501, 512, 700, 8),
    (600, 601, 400, 3, 7),
])
def test_many_rounds(n, m, landmarks, buckets, rounds):
    from parity import compare
    print("rounds", n, m, rounds, compare(_cut(n, m, 3, landmarks, buckets, rounds, 6), "lcn"), flush=True)


# a wavefront per row: more than four rounds of more than 80 entries together, or four of more than 1000
@pytest.mark.parametrize("n,m,buckets,rounds", [(900, 901, 30, 5), (899, 900, 53, 5), (901, 900, 60, 5), (70, 2100, 300, 8),
                                               (2100, 70, 3, 8), (700, 650, 5, 7), (1100, 1099, 4, 4), (9, 5000, 2, 4)])
def test_a_wavefront_per_row_in_logs(n, m, buckets, rounds):
    from parity import compare
    print("logs", n, m, buckets, rounds, compare(_cut(n, m, 4, 8, buckets, rounds, 12), "sparse"), flush=True)


# one round: a workgroup per bucket through the whole run, with 256 threads up to 6 KB a block (32 x 32), 512 up to 24 (72 x 72)
# or with more than 512 buckets, else 1024, up to 320 rows or columns a block and 160 KB (beyond either a launch per sweep);
# fewer points on a side than buckets, a single row
@pytest.mark.parametrize("mode,n,m,buckets,iters", [
    ("sparse", 32, 33, 1, 9), ("dense", 72, 72, 1, 9), ("sparse", 73, 73, 1, 9), ("sparse", 320, 100, 1, 9),
    ("dense", 100, 321, 1, 9), ("dense", 9, 320, 1, 9), ("sparse", 192, 192, 1, 9), ("sparse", 193, 193, 1, 9),
    ("dense", 1, 300, 1, 9), ("sparse", 300, 7, 40, 9), ("sparse", 2500, 2400, 90, 9), ("sparse", 4000, 4100, 33, 9),
    ("sparse", 9000, 9100, 600, 3), ("sparse", 9000, 9100, 2100, 3)])
def test_runs_bucket_by_bucket(mode, n, m, buckets, iters):
    from parity import compare
    p = _cut(n, m, 4, 8, buckets, 1, iters)
    p.b[m // 3] = 0    # a point without mass
    print("buckets", mode, n, m, buckets, compare(p, mode), flush=True)


def _in_buckets(nx, ny, iters, d=24, seed=5):
    """A problem whose cross-polytope hash puts nx[k] of X's points and ny[k] of Y's into bucket k: every point lies in
    the direction of a projection or opposite to it, whatever its length."""
    b = len(nx)
    rng = np.random.default_rng(seed)
    p = workloads.config3(n=64, d=8, landmarks=8, buckets=8, rounds=1, iters=iters, name="buckets")
    R = rng.standard_normal((d, b // 2))
    R /= np.linalg.norm(R, axis=0)

    def points(counts):
        k = rng.permutation(np.repeat(np.arange(b), counts))
        Z = R[:, k % (b // 2)].T * np.where(k < b // 2, 1.0, -1.0)[:, None] * rng.uniform(0.5, 2.0, (len(k), 1))
        return (Z + 0.002 * rng.standard_normal(Z.shape)).astype(np.float32)
    p.X, p.Y = points(nx), points(ny)
    p.a = rng.uniform(0.5, 1.5, len(p.X)).astype(np.float32)
    p.b = rng.uniform(0.5, 1.5, len(p.Y)).astype(np.float32)
    p.a /= p.a.sum()
    p.b /= p.b.sum()
    p.cost, p.lam = workloads.COST_SQEUCLID, 1.0
    p.num_buckets, p.num_rounds, p.projections = b, 1, R[None].astype(np.float32)
    for Z, counts in ((p.X, nx), (p.Y, ny)):
        assert sorted(np.bincount(oracle.crosspolytope(Z, p.projections[0], b), minlength=b)) == sorted(counts)
    return p


# blocks of unlike size: bucket by bucket with the LDS of the largest, a launch per sweep (bucket_rule.h), and with a
# block that does not fit by every choice of log_walk.h for one round; sizes that are no multiples of eight
@pytest.mark.parametrize("buckets,many,nx,ny,sx,sy", [
    (1000, 1, 190, 189, 3, 5), (2000, 7, 109, 141, 6, 3), (4096, 1, 190, 150, 1, 2), (4096, 10, 139, 141, 3, 3),
    (2000, 1, 401, 403, 6, 7), (400, 1, 499, 501, 31, 29), (200, 1, 333, 402, 21, 19), (60, 1, 401, 403, 21, 20), (2, 1, 401, 30, 30, 401)])
def test_blocks_of_unlike_size(buckets, many, nx, ny, sx, sy):
    from parity import compare
    p = _in_buckets([nx] * many + [sx] * (buckets - many), [ny] * many + [sy] * (buckets - many), 5)
    print("unlike", buckets, nx, ny, sx, sy, compare(p, "sparse", workloads.HASH_CROSSPOLYTOPE), flush=True)


def _rounds_apart(n, m, seed=5):
    """Two rounds of two buckets each: halves of both sides, then half of X's points with all of Y's (those rows' second round
    is long) and half with none (it is empty)."""
    rng = np.random.default_rng(seed)
    p = _in_buckets([n // 2, n - n // 2], [m // 2, m - m // 2], 1, d=2, seed=seed)
    p.X, p.Y = (rng.uniform(0.5, 1.5, (k, 2)) * rng.choice([-1, 1], (k, 2)) for k in (n, m))
    p.Y[:, 1] = np.abs(p.Y[:, 1])
    p.X, p.Y = p.X.astype(np.float32), p.Y.astype(np.float32)
    p.num_rounds, p.projections = 2, np.eye(2, dtype=np.float32).reshape(2, 2, 1)
    return p


# Sums out of single precision's range: the walk with running maxima, by every kernel that has one of its own.  The scalings
# before the iteration are up to e^150 off, so most rows and columns take it, and all of them have a weighty result.
@pytest.mark.parametrize("what", [
    ([41, 30, 9, 1], [37, 43, 8, 2]), ([190, 3], [189, 5]),              # bucket by bucket, no multiples of eight
    ([401, 20], [333, 45]), ([50] * 290 + [330] * 2, [49] * 292),        # one round, a launch per sweep
    (3000, 2999, 700, 2), (1500, 1499, 40, 3), (1200, 1201, 60, 4),      # two to four, flat
    (700, 661, "apart"), (8101, 407, "apart"),                           # two, round by round; an empty round
    (1000, 999, 60, 5), (700, 650, 5, 7)])                               # more, flat, a wavefront per row
def test_sums_out_of_range(what):
    import torch
    import paper_2107_06876_amd as lcn
    from parity import gpu_build
    hash_kind = workloads.HASH_CROSSPOLYTOPE
    if isinstance(what[0], list):
        p = _in_buckets(what[0], what[1], 1)
    elif what[-1] == "apart":
        p = _rounds_apart(what[0], what[1])
    else:
        p, hash_kind = _cut(what[0], what[1], 4, 8, what[2], what[3], 1), workloads.HASH_KMEANS
        p.lam = 40.0
    B = oracle.build_problem(p.X, p.Y, p.cost, p.lam, "sparse", p.num_landmarks, p.landmark_seed, p.kmeans_iters, p.ridge, hash_kind,
                             p.num_buckets, p.num_rounds, p.lsh_seed, p.projections, branching=p.branching, and_width=p.and_width)
    rng = np.random.default_rng(3)
    log_u, log_v = (rng.uniform(-150.0, 150.0, k).astype(np.float32) for k in (len(p.X), len(p.Y)))
    h = gpu_build(p, "sparse", hash_kind)
    lcn.lcn_set_scalings(h, torch.from_numpy(log_u).cuda(), torch.from_numpy(log_v).cuda())
    lcn.sinkhorn_run(h, 1, check=False)
    got = [v.cpu().numpy().astype(np.float64) for v in lcn.lcn_get_scalings(h)]
    lcn.lcn_destroy(h)
    rows, cols, logs = np.repeat(np.arange(len(p.X)), np.diff(B.op.rowptr)), B.op.colidx, np.log(B.op.val)

    def logsumexp(at, terms, size):
        top = np.full(size, -np.inf)
        np.maximum.at(top, at, terms)
        total = np.zeros(size)
        np.add.at(total, at, np.exp(terms - top[at]))
        with np.errstate(divide="ignore"):
            return top + np.log(total)
    with np.errstate(divide="ignore", invalid="ignore"):
        want_u = np.log(p.a.astype(np.float64)) - logsumexp(rows, logs + log_v.astype(np.float64)[cols], len(p.X))
        want_v = np.log(p.b.astype(np.float64)) - logsumexp(cols, logs + want_u[rows], len(p.Y))
    beyond, least = 0, min(len(p.X), len(p.Y)) // 4
    for g, w, before in ((got[0], want_u, log_u), (got[1], want_v, log_v)):
        some = np.isfinite(w)
        assert (g[~some] == -np.inf).all()
        # What is returned is rounded to single precision, 2^-17 below 256.  Where the first walk does, its terms are
        # exp(k + (p - shift)) of numbers below 70: the difference, the sum and the product with log2(e) are rounded to 2^-18
        # each, k and exp to 2^-21; log v takes log u's error on top of its own.
        assert np.abs(w[some]).max() < 256 and np.abs(g[some] - w[some]).max() <= 2.0 ** -17 + 2 * (3 * 2.0 ** -18 + 2.0 ** -20)
        beyond += int((np.abs(before[some] - w[some]) > 70).sum())   # sum over shift: exp of that, and 1e30 is e^69
    assert beyond >= least


def test_a_run_bucket_by_bucket_in_parts():
    """The state passes through memory between the launches of a run (4 ms each, some 2000 iterations) and between runs without a loss."""
    import torch
    import paper_2107_06876_amd as lcn
    from parity import gpu_build
    got = []
    for runs in ([4100], [4, 4096], [1000, 3100]):
        h = gpu_build(_cut(40, 41, 4, 8, 3, 1, 1), "sparse")
        for iters in runs:
            lcn.sinkhorn_run(h, iters)
        got.append(lcn.lcn_get_scalings(h) + (lcn.transport_cost(h),))
        lcn.lcn_destroy(h)
    for other in got[1:]:
        assert torch.equal(got[0][0], other[0]) and torch.equal(got[0][1], other[1]) and got[0][2] == other[2]


# a query in logs: up to 2^22 entries by 512 workgroups, above that by up to 2048, fewer where rows run out
@pytest.mark.parametrize("n,m,buckets", [(8300, 8301, 8), (8300, 8301, 40), (1800, 1801, 1), (20000, 300, 1)])
def test_queries_over_many_rows(n, m, buckets):
    import torch
    import paper_2107_06876_amd as lcn
    from parity import compare, gpu_build
    p = _cut(n, m, 3, 8, buckets, 1, 4)
    print("query", n, m, buckets, compare(p, "sparse"), flush=True)
    # what the library asks for beforehand, told how many pairs there are, is enough
    h = gpu_build(p, "sparse")
    info = lcn.lcn_get_info(h)
    lsh = dict(num_buckets=buckets, num_rounds=1, kmeans_iters=p.kmeans_iters, seed=1)
    assert lcn.lcn_workspace_bytes(n, m, 3, lcn.MODE_SPARSE, None, lsh, nnz_guess=info.nnz_stored) >= info.workspace_used
    lcn.lcn_destroy(h)


@pytest.mark.parametrize("n,m,d,landmarks,buckets,rounds", [
    (4096, 4096, 5, 17, 33, 2),      # exactly one range of points, bucket arrays on multiples of four
    (4099, 4094, 5, 17, 33, 3),      # one point more, bucket arrays off by one, two and three
    (8193, 8193, 40, 64, 300, 2),    # three ranges, more than 256 clusters
    (3, 4, 2, 3, 5, 2),              # fewer points than a group of four has room for
    (900, 801, 530, 20, 12, 1),      # rows too long for sums in registers
    (9001, 9002, 3, 40, 3800, 1),    # clusters times points above the limit: counting sort
    (70000, 70001, 2, 30, 60, 1),    # too many points to advance together: a stream per run
    (5000, 5003, 512, 70, 9, 1),     # the widest rows summed in registers
])
def test_kmeans_ranges_and_runs(monkeypatch, n, m, d, landmarks, buckets, rounds):
    """Landmarks and buckets equal those of the exact rule applied to every point, which shares neither the filter nor
    the list of undecided points."""
    import torch
    import paper_2107_06876_amd as lcn
    from parity import gpu_build
    p = _cut(n, m, d, landmarks, buckets, rounds, 1, kmeans_iters=4)
    p.X[: n // 5] = p.X[0]   # coinciding points: ties, and a cluster far larger than the others
    got = {}
    for exact in ("0", "1"):
        monkeypatch.setenv("LCN_EXACT_ASSIGN_ONLY", exact)
        h = gpu_build(p, "lcn")
        got[exact] = (lcn.lcn_get_landmarks(h), lcn.lcn_get_buckets(h))
        lcn.lcn_destroy(h)
    assert torch.equal(got["0"][0], got["1"][0]) and torch.equal(got["0"][1], got["1"][1])


# runs together up to 2^14 points and 64 landmarks (few scores), up to 2^15 or as two runs (very few), as more rounds than
# lanes; otherwise each on its own.  Centroids by members up to 2^26 clusters times points of all runs, twice that with
# more rounds than lanes, always up to 2^14 points
@pytest.mark.parametrize("n,m,d,landmarks,buckets,rounds", [
    (8192, 8192, 130, 64, 100, 2),   # the most points that advance together
    (8192, 8193, 130, 64, 100, 2),   # one point more
    (8192, 8192, 5, 65, 33, 2),      # one landmark more
    (8000, 7999, 130, 64, 300, 2),   # few points, many scores
    (16384, 16384, 5, 64, 33, 2),    # very few scores
    (16384, 16385, 5, 64, 33, 2),    # ... and one point more
    (16384, 16385, 5, 64, 33, 1),    # the same, two runs
    (3000, 3001, 40, 70, 50, 4),     # more rounds than lanes
    (20000, 20001, 3, 20, 300, 5),
    (20000, 20000, 3, 20, 700, 5),   # ... above 2^27: sorted
    (10000, 10000, 3, 1, 1118, 3),   # just below 2^26
    (10000, 10000, 3, 2, 1118, 3),   # just above: sorted
    (8000, 8000, 3, 5, 1500, 3),     # few points: by members all the same
    (400, 390, 640, 64, 65, 2),      # rows of more than 512 dimensions: 64 centroids at a time, 256
    (400, 390, 515, 3, 64, 1),       # ... and a last piece of three dimensions
])
def test_runs_together_or_apart(monkeypatch, n, m, d, landmarks, buckets, rounds):
    test_kmeans_ranges_and_runs(monkeypatch, n, m, d, landmarks, buckets, rounds)


@pytest.mark.parametrize("n,m,d,landmarks,buckets,rounds", [
    (8192, 8193, 130, 64, 100, 2), (3000, 3001, 40, 70, 50, 3), (3000, 3001, 40, 70, 50, 5), (70000, 70001, 2, 30, 60, 1),
    (10000, 10000, 3, 2, 1118, 3),
])
def test_runs_without_streams_of_their_own(monkeypatch, n, m, d, landmarks, buckets, rounds):
    monkeypatch.setenv("LCN_BUILD_OVERLAP", "0")
    test_kmeans_ranges_and_runs(monkeypatch, n, m, d, landmarks, buckets, rounds)


def test_undecided_points_are_those_of_the_last_run():
    """What lcn_get_info reports belongs to the last hash round, however the runs advance: together, each on its own, with
    and without landmarks beside them."""
    import paper_2107_06876_amd as lcn
    from parity import gpu_build
    p = _cut(3000, 3001, 7, 64, 40, 3, 1, kmeans_iters=3)
    p.X, p.Y = np.round(2 * p.X).astype(np.float32), np.round(2 * p.Y).astype(np.float32)   # ties
    got = []
    for mode, landmarks, rounds in (("lcn", 64, 3), ("lcn", 65, 3), ("sparse", 64, 3), ("lcn", 64, 2), ("sparse", 64, 2)):
        p.num_landmarks, p.num_rounds = landmarks, rounds
        h = gpu_build(p, mode)
        got.append(lcn.lcn_get_info(h).undecided_last)
        lcn.lcn_destroy(h)
    assert got[0] == got[1] == got[2] > 0 and got[3] == got[4] > 0


def test_hierarchical_levels_by_members_and_sorted():
    """Three levels of 15, 225 and 3600 clusters: the last has too many for 20 001 points to be updated by members."""
    from parity import compare
    p = _cut(10000, 10001, 3, 8, 3600, 1, 4)
    p.branching = (15, 15, 16)
    print("hierarchical", compare(p, "sparse"), flush=True)


@pytest.mark.parametrize("members", [1, 15, 16, 17, 33, 48, 63, 64, 65, 130])
def test_pieces_of_a_tile(members):
    """Sparse values and their derivatives where a bucket holds so many points of one side and 20 of the other: pieces
    of 16 x 16 dealt to four wavefronts.  A single bucket, so that the sizes are exact."""
    import torch
    import paper_2107_06876_amd as lcn
    from parity import compare, gpu_build
    p = _cut(members, 20, 5, 4, 1, 1, 10)
    print("pieces", members, compare(p, "lcn"), flush=True)
    p.X, p.Y, p.a, p.b = p.Y, p.X, p.b, p.a
    print("pieces", members, compare(p, "lcn"), flush=True)
    h = gpu_build(p, "lcn")
    lcn.sinkhorn_run(h, 10)
    rowptr, cols, _ = lcn.lcn_get_csr(h)
    gU, gWt, gsp, gnys = lcn.lcn_backward(h, nnz=len(cols))
    # one bucket: the pattern is everything, and with a_i b_j mass the derivative of every K^sp entry is -lambda u_i v_j
    log_u, log_v = (t.double() for t in lcn.lcn_get_scalings(h))
    K = torch.exp(-((torch.from_numpy(p.X).double()[:, None] - torch.from_numpy(p.Y).double()[None]) ** 2).sum(2) / p.lam)
    want = -p.lam * torch.exp(log_u.cpu()[:, None] + log_v.cpu()[None]) * K
    got = gsp.cpu().double().reshape(want.shape)
    # scalings in single precision (their logs to 6e-8 of up to about 10) and one rounding of the product
    assert float((got - want).abs().max()) <= 4e-6 * float(want.abs().max())
    lcn.lcn_destroy(h)


@pytest.mark.parametrize("total,d", [(1, 1), (255, 31), (256, 32), (257, 33), (1000, 100)])
def test_deletion_costs_sizes(total, d):
    import torch
    import paper_2107_06876_amd as lcn
    rng = np.random.default_rng(total + d)
    X, alpha = rng.standard_normal((total, d)).astype(np.float32), rng.random(d).astype(np.float32)
    got = lcn.lcn_deletion_costs(torch.from_numpy(X).cuda(), torch.from_numpy(alpha).cuda()).cpu().numpy()
    np.testing.assert_array_equal(got, oracle.deletion_costs(X, alpha))


def test_many_batches_at_once():
    """More batch handles alive than pinned blocks are kept, given back in another order, from several threads and
    streams: each keeps its own results."""
    import threading
    import torch
    import paper_2107_06876_amd as lcn
    rng = np.random.default_rng(3)

    def batch(pairs, seed):
        r = np.random.default_rng(seed)
        x_off = np.concatenate([[0], np.cumsum(r.integers(5, 40, pairs))]).astype(np.int64)
        y_off = np.concatenate([[0], np.cumsum(r.integers(5, 40, pairs))]).astype(np.int64)
        X = torch.from_numpy(r.standard_normal((x_off[-1], 8)).astype(np.float32)).cuda()
        Y = torch.from_numpy(r.standard_normal((y_off[-1], 8)).astype(np.float32)).cuda()
        return X, Y, x_off, y_off, np.full(pairs, 2.0, dtype=np.float32)

    def solve(args, stream=None):
        h = lcn.lcn_build_batched(*args, lcn.COST_SQEUCLID, lcn.MODE_DENSE, stream=stream)
        lcn.sinkhorn_run(h, 20)
        return h

    problems = [batch(int(rng.integers(1, 50)) if i else 9000, 100 + i) for i in range(12)]
    want = []
    for args in problems:
        h = solve(args)
        want.append(lcn.lcn_batched_results(h))
        lcn.lcn_destroy(h)
    handles = [solve(args) for args in problems]
    for i in rng.permutation(len(problems)):
        got = lcn.lcn_batched_results(handles[i])
        np.testing.assert_array_equal(got[0], want[i][0])
        np.testing.assert_array_equal(got[1], want[i][1])
        lcn.lcn_destroy(handles[i])
    torch.cuda.synchronize()
    wrong = []

    def work(mine):
        s = torch.cuda.Stream()
        for i in mine:
            h = solve(problems[i], stream=s.cuda_stream)
            got = lcn.lcn_batched_results(h)
            if not (np.array_equal(got[0], want[i][0]) and np.array_equal(got[1], want[i][1])):
                wrong.append(i)
            lcn.lcn_destroy(h)

    threads = [threading.Thread(target=work, args=([i for i in range(12) if i % 4 == t],)) for t in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong


@pytest.mark.parametrize("n,m,blocks", [
    (7, 1, [(0, 7)]), (5, 63, [(4, 1), (0, 3)]), (9, 1023, [(0, 9), (1, 5)]), (17, 1024, [(0, 16), (13, 4)]),
    (18, 1025, [(0, 18), (16, 2)]), (33, 2049, [(0, 33), (3, 17)]), (1, 5000, [(0, 1)]),
])
def test_dense_plan_blocks(n, m, blocks):
    """Four rows and 1024 columns per wavefront: every entry of a block is written, none beside it.  Against the stored
    kernel: the logs of the scalings come rounded to single precision, and so do the kernel's and the plan's values."""
    import torch
    import paper_2107_06876_amd as lcn
    from parity import gpu_build
    p = _cut(n, m, 3, 0, 0, 0, 4)
    p.a[0] = 0.0    # a row without mass
    h = gpu_build(p, "dense")
    lcn.sinkhorn_run(h, 4)
    lu, lv = (x.double() for x in lcn.lcn_get_scalings(h))
    K = lcn.lcn_get_csr(h)[2].double().reshape(n, m)
    t = lu[:, None] + lv[None, :]
    want = K * torch.exp(t)
    bound = want * 2.0 ** -24 * (2 + 1.01 * torch.nan_to_num(lu[:, None].abs() + lv[None, :].abs(), posinf=0.0)) + 1e-37
    for i0, rows in blocks:
        room = torch.full((rows * m + 64,), -7.0, device=h.device)
        lcn.lcn_plan_rows(h, i0, rows, out=room[:rows * m].view(rows, m))
        got = room[:rows * m].view(rows, m).double()
        assert bool((room[rows * m:] == -7.0).all())
        assert bool(((got - want[i0:i0 + rows]).abs() <= bound[i0:i0 + rows]).all()), (i0, rows)
    lcn.lcn_destroy(h)


@pytest.mark.parametrize("landmarks", [5, 40, 300])
def test_a_given_centroid_that_is_not_a_number(monkeypatch, landmarks):
    """The exact rule keeps the first of the centroids that no other beats, and nothing beats a distance that is not a
    number: with such a centroid in front every point is its member.  The filter decides nothing then."""
    import torch
    import paper_2107_06876_amd as lcn
    rng = np.random.default_rng(5)
    X = torch.from_numpy(rng.standard_normal((400, 6)).astype(np.float32)).cuda()
    Y = torch.from_numpy(rng.standard_normal((300, 6)).astype(np.float32)).cuda()
    a, b = torch.full((400,), 1 / 400, device="cuda"), torch.full((300,), 1 / 300, device="cuda")
    start = torch.cat([X, Y])[:landmarks].clone()
    start[0] = float("nan")
    got = {}
    for exact in ("0", "1"):
        monkeypatch.setenv("LCN_EXACT_ASSIGN_ONLY", exact)
        lm = dict(num_landmarks=landmarks, kmeans_iters=1, seed=1, init=lcn.INIT_GIVEN, init_centroids=start, ridge=1e-3)
        h = lcn.lcn_build(X, Y, a, b, 4.0, lcn.COST_SQEUCLID, lcn.MODE_NYSTROM, landmarks=lm)
        got[exact] = lcn.lcn_get_landmarks(h)
        lcn.lcn_destroy(h)
    assert torch.equal(got["0"], got["1"])
    assert torch.equal(got["0"][1:], start[1:])
    # one rounding of the mean to single precision, and sums in units of 2^-32
    assert float((got["0"][0].double() - torch.cat([X, Y]).double().mean(0)).abs().max()) < 1e-7
