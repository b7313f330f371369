// Many small transport problems in one launch (the graph-pair workloads of
// Sec. 6): one workgroup per pair, everything in LDS.
//
// Build: the same method as the large path, per pair -- k-means landmarks and
// k-means LSH buckets on X_p u Y_p by the exact bucket rule, Nystrom factors in
// fp64, exact kernel values on pairs that share a bucket (Secs. 3-4).  At these
// sizes (at most 64 points per side) the approximated kernel K~ = U A^{-1} V +
// (K^sp - K^sp_Nys) is written out as a dense 64 x 64 fp32 tile, which is what
// the iteration then keeps in registers.
//
// Iteration: Sinkhorn on the bipartite-matching matrix of Sec. 6,
//   K_BP = [[K~, diag(k_p,eps)], [diag(k_eps,q), 1]],
// using its block formulas (only the two diagonals are stored), with the
// log-sum-exp max-shift taken out per vector (App. "Implementational details").
// Without deletion costs it is plain Sinkhorn on K~.
//
// Compiled with -ffp-contract=off: the bucket rule needs separate multiply and add.
#include <cmath>
#include <cstring>
#include <mutex>
#include <new>
#include <type_traits>

#include "iter_common.h"   // cross-lane sums and maxima through the DPP data path
#include "lcn_internal.h"

#pragma clang fp contract(off)

namespace lcn {

constexpr int BMAX = 64;   // points per side
constexpr int BD = 64;     // dimensions
constexpr int BL = 16;     // landmarks, buckets
constexpr int BR = 4;      // hash rounds
constexpr uint32_t BATCH_MAGIC = 0x4C434E42u;  // "LCNB"

struct BatchDev {
    int P, d, cost, mode, l, b, R, T_l, T_b, bp;
    int max_points;               // n + m of the largest pair
    unsigned row4;                // first centroid row of every k-means run, in fours, six bits each (see build_rows)
    int mt;                       // tiles of 16 rows they fill
    unsigned long long seed_l, seed_b;
    double ridge;
    const float *X, *Y;           // caller's points (fp32 copies in the workspace)
    const long long *x_off, *y_off;
    const float *lambda;
    const float *del_x, *del_y;   // deletion costs or null
    float *Kt;                    // [P][64][64]
    double *kpe, *keq;            // exp(-del / lambda)
    float *landmarks;             // [P][l][d]
    int *buckets;                 // per pair [R][n_p + m_p], pairs back to back at R * (x_off + y_off)
    double *log_u, *log_v;        // per pair at x_off + y_off, length n + m each (n resp. m without BP)
    float *row_marg, *col_marg;   // marginals of the last run's plan, laid out like log_u and log_v (null: no room)
    double *dist, *resid;         // [P], host memory
    unsigned long long *counters; // [0] non-positive sums, [1] / [2] sums of exactly zero without signed terms (rows / columns), per sweep
    int *marks;                   // host memory: [0] a landmark matrix is not positive definite, [1] some counter is not zero
};

__device__ inline unsigned long long splitmix64_dev(unsigned long long &state)
{
    unsigned long long z = (state += 0x9E3779B97F4A7C15ULL);
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ULL;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBULL;
    return z ^ (z >> 31);
}

typedef double double4_t __attribute__((ext_vector_type(4)));
typedef float float4_t __attribute__((ext_vector_type(4)));
typedef int int4_t __attribute__((ext_vector_type(4)));

// The centroids of all k-means runs of a pair (run 0: the landmarks if there are any, then the hash rounds)
// share tiles of 16 rows; a run starts on a multiple of four and does not straddle tiles.
__host__ inline void build_rows(BatchDev &D)
{
    int row = 0, q = 0;
    D.row4 = 0u;
    auto put = [&](int k) {
        const int k4 = (k + 3) & ~3;
        if (row % 16 + k4 > 16) row = (row + 15) & ~15;
        D.row4 |= (unsigned)(row / 4) << 6 * q++;
        row += k4;
    };
    if (D.l > 0) put(D.l);
    for (int r = 0; r < D.R; ++r) put(D.b);
    D.mt = (row + 15) / 16;
}

// Entries of a pair's kernel that share a bucket and are still to be formed, a wavefront's: dot products and places.
struct NearList {
    double dot[128];
    unsigned short place[128];   // 64 i + j
};

// LDS of the build kernel, sized by the batch (its d, l, buckets, rounds and largest pair), not by the
// upper limits: doubles first, then floats, then integers.
struct BuildLds {
    int zs, ls, rows;   // row length of points / centroids and of the factors; points of the largest pair
    size_t f, am, sums, pn, rn, z, cent, mid, assign, cnts, start, flags, bytes;
};

// dt: tiles of 16 dimensions, waves: wavefronts of the workgroup
__host__ __device__ inline BuildLds build_lds(int l, int runs, int mt, int dt, int max_points, int waves)
{
    BuildLds L;
    // rows of 16-byte pieces, an odd number of them: the operand reads of a wavefront then spread over the banks
    L.zs = 16 * dt + 4;
    L.ls = l + 1 + (l & 1);   // odd, for the same reason
    L.rows = (max_points + 15) & ~15;
    size_t at = 0;
    auto take = [&](size_t bytes) {
        const size_t here = at;
        at += (bytes + 15) & ~(size_t)15;
        return here;
    };
    // the member sums are done with when the factors are formed: they share their place
    const size_t f_bytes = l > 0 ? sizeof(double) * L.rows * L.ls : 0, sum_bytes = sizeof(double) * mt * dt * 256;
    L.f = L.sums = take(f_bytes > sum_bytes ? f_bytes : sum_bytes);
    L.am = take(sizeof(double) * l * (l + 1));
    L.pn = take(sizeof(double) * L.rows);
    L.rn = take(sizeof(double) * BL);
    L.z = take(sizeof(float) * L.rows * L.zs);
    // (when the kernel's values are formed the centroids are done with, and every wavefront has its NearList there)
    const size_t cent_bytes = sizeof(float) * 16 * mt * L.zs, list_bytes = sizeof(NearList) * waves;
    L.cent = take(cent_bytes > list_bytes ? cent_bytes : list_bytes);
    L.mid = take(sizeof(float) * 16 * dt);
    L.assign = take(runs * L.rows + 112);   // bytes; 128 of a run are read whatever the number of points
    L.cnts = take(sizeof(int) * 2 * 16 * mt);
    L.start = take(2 * sizeof(int) * 16 * mt);
    L.flags = take(sizeof(int) * 8);
    L.bytes = at;
    return L;
}

// Cost of two points from their dot product and squared norms a2, b2, for an entry of the kernel.  Where the norms
// nearly cancel (squared distance below 1e-4 of their sum) it is taken from the differences of the points' rows (LDS,
// zero padded to dp dimensions) instead; coinciding points are at distance zero exactly.  The cost's relative error is
// about 1e-12 then and below 1.5e-10 in any case, the entry's (an exponent above -104) below 1.6e-8, a quarter of its
// rounding to single precision.
__device__ inline double cost_of_dot(double dot, double a2, double b2, const float *x, const float *y, int dp, int cost)
{
    if (cost == LCN_COST_COSINE) return 1.0 - dot / (sqrt(a2) * sqrt(b2));
    double sq = fma(-2.0, dot, a2 + b2);
    if (!(sq > 1e-4 * (a2 + b2))) {
        sq = 0.0;
        for (int k = 0; k < dp; ++k) {
            const double t = (double)x[k] - (double)y[k];
            sq = fma(t, t, sq);
        }
    }
    return cost == LCN_COST_EUCLID ? sqrt(sq) : sq;
}

// the smaller of two numbers in one instruction (fminf first quiets both arguments)
__device__ inline float min32(float a, float b)
{
    float r;
    asm("v_min_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

// over the four lanes that share l % 16
__device__ inline float quarter_min(float v)
{
    const auto a = __builtin_amdgcn_permlane32_swap(__float_as_int(v), __float_as_int(v), false, false);
    v = min32(__int_as_float(a[0]), __int_as_float(a[1]));
    const auto b = __builtin_amdgcn_permlane16_swap(__float_as_int(v), __float_as_int(v), false, false);
    return min32(__int_as_float(b[0]), __int_as_float(b[1]));
}

__device__ inline float quarter_sum(float v)
{
    const auto a = __builtin_amdgcn_permlane32_swap(__float_as_int(v), __float_as_int(v), false, false);
    v = __int_as_float(a[0]) + __int_as_float(a[1]);
    const auto b = __builtin_amdgcn_permlane16_swap(__float_as_int(v), __float_as_int(v), false, false);
    return __int_as_float(b[0]) + __int_as_float(b[1]);
}

__device__ inline double quarter_sum(double v)
{
    double w = v;
    lane_swap<32>(v, w);
    v += w;
    w = v;
    lane_swap<16>(v, w);
    return v + w;
}

__device__ inline unsigned quarter_or(unsigned v)
{
    const auto a = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    v = a[0] | a[1];
    const auto b = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    return b[0] | b[1];
}

// Cholesky factor of the l x l matrix A (LDS), l <= LP, by one wavefront, lane i holding row i: L below the
// diagonal in place, 1 / L_jj behind the matrix.
template <int LP>
__device__ inline void landmark_cholesky(double *A, int l, int *not_positive)
{
    const int lane = threadIdx.x & 63;
    double a[LP];
#pragma unroll
    for (int k = 0; k < LP; ++k) a[k] = (lane < l && k < l) ? A[lane * l + k] : (lane == k ? 1.0 : 0.0);
    double rdiag = 1.0;
    bool bad = false;
#pragma unroll
    for (int j = 0; j < LP; ++j) {
        double dd = lane_value(a[j], j);
        if (!(dd > 0.0)) {
            bad = true;
            dd = 1.0;
        }
        double rs = __builtin_amdgcn_rsq(dd);   // 1 / sqrt to fp64 rounding: estimate and two Newton steps
        rs = fma(0.5 * rs, fma(-dd * rs, rs, 1.0), rs);
        rs = fma(0.5 * rs, fma(-dd * rs, rs, 1.0), rs);
        rdiag = lane == j ? rs : rdiag;
        a[j] *= rs;
#pragma unroll
        for (int k = j + 1; k < LP; ++k) a[k] = fma(-a[j], lane_value(a[j], k), a[k]);
    }
    if (bad && lane == 0) *not_positive = 1;
#pragma unroll
    for (int k = 0; k < LP; ++k)
        if (lane < l && k < lane) A[lane * l + k] = a[k];
    if (lane < l) A[l * l + lane] = rdiag;
}

// One workgroup of NT threads builds a pair; everything is in LDS.  What bounds it is latency: barriers,
// chains of dependent operations on a few dozen points, and a vector instruction every 6.8 clocks where
// a SIMD has one wavefront only (4.5 with several).  So
//  * all k-means runs of the pair (landmarks and every hash round) advance together, a Lloyd iteration
//    costing three barriers however many runs there are, and stop as soon as no assignment changed
//    (from then on an iteration reproduces its own centroids bit for bit);
//  * an assignment is a product on the fp32 matrix instruction, |c|^2 - 2 z.c for 16 points (columns; their
//    operands stay in registers for all iterations) against 16 centroid rows: centroids within 2 delta of a
//    point's smallest score are its candidates, and only a point with several of them (near ties) is decided
//    by the bucket rule itself;
//  * the member sums are products as well, of the 0/1 membership matrix with the digits of the fixed-point values
//    on the 8-bit matrix instruction: whole numbers, so exact in any order;
//  * the start indices of a run are drawn by a lane each and the shuffle is resolved by ballots;
//  * the Nystrom values are products of L^{-1} u and L^{-1} v (A = L L^T): a Cholesky by one wavefront in
//    registers and one forward substitution per point, no inverse;
//  * the costs of the pairs that share a bucket come from dot products on the matrix instruction (see
//    cost_of_dot), and so do the Nystrom values; tiles of the kernel without such a pair skip the costs.
// Pairs of 16 to 64 points (d = 32, l = 8, b = 4, ten Lloyd iterations): the kernel takes 37 us for 16 pairs, 86 us for 1024
// and 276 us for 4096 (43, 115 and 363 with scores and member sums on v_mfma_f64_16x16x4, whose instruction takes four
// times the matrix cores' time for an eighth of the dimensions of scores, or a sixteenth of the points of sums).
// Layout of v_mfma_f64_16x16x4_f64: lane l gives A[l % 16][l / 16] and B[l / 16][l % 16] and receives
// D[4 v + l / 16][l % 16], v = 0..3 (of the 32-bit instructions D[4 (l / 16) + v][l % 16]); which dimension a step of a dot product takes is free, so a lane reads
// four consecutive ones (16 t + 4 (l / 16) ..) for four steps.
template <int NT, int DT>
__global__ __launch_bounds__(NT, 4) void batched_build_kernel(BatchDev B)
{
    constexpr int NW = NT / 64, TPW = 8 / NW;   // wavefronts; tiles of 16 points each of them holds (at most 128 points)
    extern __shared__ __align__(16) unsigned char lds[];
    const int l = B.l, d = B.d, runs = (l > 0 ? 1 : 0) + B.R;
    const BuildLds L = build_lds(l, runs, B.mt, DT, B.max_points, NW);
    constexpr int zs = 16 * DT + 4;
    double *F = (double *)(lds + L.f), *Am = (double *)(lds + L.am), *sums = (double *)(lds + L.sums);
    double *pn = (double *)(lds + L.pn), *rn = (double *)(lds + L.rn);   // squared norms of the points, of the landmarks
    float *Z = (float *)(lds + L.z), *cent = (float *)(lds + L.cent), *mid = (float *)(lds + L.mid);
    unsigned char *assign = lds + L.assign;
    int *cnts = (int *)(lds + L.cnts), *start = (int *)(lds + L.start);
    int *owner = start + 16 * B.mt;   // of every centroid row: 256 run + index in the run, -1 if none
    // [0], [1]: some assignment changed (by parity); [2]: not positive definite; [3]: a large coordinate;
    // [4:5]: bits of the largest squared norm of a point; [6]: a coordinate the rule alone decides on
    int *flags = (int *)(lds + L.flags);

    const int p = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 15, quarter = lane >> 4;
    const long long x0 = B.x_off[p], y0 = B.y_off[p];
    const int n = (int)(B.x_off[p + 1] - x0), m = (int)(B.y_off[p + 1] - y0);
    const int N = n + m, PT = (N + 15) / 16, rows16 = 16 * B.mt;
    const double lam = (double)B.lambda[p];
    const bool low_rank = l > 0, hashed = B.R > 0;
    const int first_hash = low_rank ? 1 : 0;
    const int buckets = B.b;
    auto k_of = [&](int q) { return q < first_hash ? l : buckets; };
    const int T_l = B.T_l, T_b = B.T_b;
    auto iters_of = [&](int q) { return q < first_hash ? T_l : T_b; };
    const unsigned row4 = B.row4;
    auto row_of = [&](int q) { return (int)(row4 >> 6 * q & 63u) * 4; };
    const int landmark_rows = (l + 3) & ~3;

    if (tid < 8) flags[tid] = 0;
    for (int e = tid; e < 2 * rows16; e += NT) cnts[e] = 0;
    for (int e = tid; e < rows16; e += NT) owner[e] = start[e] = -1;   // rows that hold no centroid
    __syncthreads();
    // the pair's points, X then Y, zero padded to whole tiles of points and dimensions
    {
        constexpr int LANES = 16 * DT, STEP = NT / LANES;
        const int r0 = tid / LANES, j = tid % LANES;
        bool large = false, beyond = false;
#pragma unroll 4
        for (int i = r0; i < 16 * PT; i += STEP) {
            const float *src = i < n ? B.X + (x0 + i) * d : B.Y + (y0 + i - n) * d;
            const float v = (i < N && j < d) ? src[j] : 0.f;
            Z[i * zs + j] = v;
            large = large || !(fabsf(v) < 8192.f);
            beyond = beyond || !(fabsf(v) < 16777216.f);
        }
        if (large) flags[3] = 1;
        if (beyond) flags[6] = 1;
    }
    // Start of a run: the first k slots of a Fisher-Yates shuffle of 0 .. N-1 driven by splitmix64.  Lane t
    // draws j_t; slot t receives what slot j_t holds, which is its own index unless an earlier step
    // s swapped there (the last such s counts: slot j_s received slot s's value V_s).
    for (int q = wave; q < runs; q += NW) {
        const bool lm = q < first_hash;
        const int k = k_of(q);
        unsigned long long state = (lm ? B.seed_l + (unsigned long long)p
                                       : B.seed_b + (unsigned long long)p * B.R + (unsigned long long)(q - first_hash)) +
                                   (unsigned long long)lane * 0x9E3779B97F4A7C15ULL;
        const unsigned long long r = splitmix64_dev(state);
        const int J = lane < k ? lane + (int)(r % (unsigned long long)(N - lane)) : -1;
        int V = lane, pick = 0;
        for (int t = 0; t < k; ++t) {
            const int jt = __builtin_amdgcn_readlane(J, t);
            const unsigned long long below = (1ull << t) - 1ull;
            const unsigned long long at_t = __ballot(J == t) & below, at_j = __ballot(J == jt) & below;
            const int vt = at_t ? __builtin_amdgcn_readlane(V, 63 - __builtin_clzll(at_t)) : t;
            const int vj = at_j ? __builtin_amdgcn_readlane(V, 63 - __builtin_clzll(at_j)) : jt;
            if (lane == t) {
                V = vt;
                pick = jt == t ? vt : vj;
            }
        }
        if (lane < k) {
            start[row_of(q) + lane] = pick;
            owner[row_of(q) + lane] = 256 * q + lane;
        }
    }
    __syncthreads();
    for (int e = tid; e < 16 * DT * rows16; e += NT) {
        const int c = e / (16 * DT), j = e % (16 * DT), s = start[c];
        cent[c * zs + j] = s >= 0 ? Z[s * zs + j] : 0.f;
    }
    // the scores are formed about the middle of eight points, wherever the pair lies
    if (B.mt > 0 && tid < 16 * DT) {
        float s = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) s += Z[(e * N >> 3) * zs + tid];
        mid[tid] = 0.125f * s;
    }
    if (B.mt > 0) __syncthreads();
    for (int e = tid; e < 256 * B.mt * DT; e += NT) sums[e] = 0.0;
    // this wavefront's points less the middle as matrix operands; squared norms of the points
    float zop[TPW][4 * DT], mid_sq = 0.f;
    if (B.mt == 0) {   // no k-means run: the norms are all
#pragma unroll
        for (int u = 0; u < TPW; ++u) {
            const int pt = 16 * (wave + NW * u) + col;
            if (pt >= 16 * PT) continue;   // the same in every lane
            double sq = 0.0;
#pragma unroll
            for (int t = 0; t < DT; ++t) {
                const float4 v = *(const float4 *)(Z + pt * zs + 16 * t + 4 * quarter);
                const float f[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                for (int e = 0; e < 4; ++e) sq = fma((double)f[e], (double)f[e], sq);
            }
            sq = quarter_sum(sq);
            if (quarter == 0) pn[pt] = sq;
        }
    } else {
        float about[4 * DT];
#pragma unroll
        for (int t = 0; t < DT; ++t) {
            const float4 v = *(const float4 *)(mid + 16 * t + 4 * quarter);
            about[4 * t] = v.x, about[4 * t + 1] = v.y, about[4 * t + 2] = v.z, about[4 * t + 3] = v.w;
        }
#pragma unroll
        for (int e = 0; e < 4 * DT; ++e) mid_sq = fmaf(about[e], about[e], mid_sq);
        mid_sq = quarter_sum(mid_sq);
        double largest = 0.0;
#pragma unroll
        for (int u = 0; u < TPW; ++u) {
            const int pt = 16 * (wave + NW * u) + col;
            double sq = 0.0, sq_about = 0.0;
#pragma unroll
            for (int t = 0; t < DT; ++t) {
                float4 v = {0.f, 0.f, 0.f, 0.f};
                if (pt < 16 * PT) v = *(const float4 *)(Z + pt * zs + 16 * t + 4 * quarter);
                const float f[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float z = f[e] - about[4 * t + e];
                    zop[u][4 * t + e] = z;
                    sq = fma((double)f[e], (double)f[e], sq);
                    sq_about = fma((double)z, (double)z, sq_about);
                }
            }
            sq = quarter_sum(sq);
            sq_about = quarter_sum(sq_about);
            if (quarter == 0 && pt < 16 * PT) pn[pt] = sq;
            largest = fmax(largest, pt < N ? sq_about : 0.0);
        }
        largest = wave_max(largest);
        if (lane == 0) atomicMax((unsigned long long *)(flags + 4), (unsigned long long)__double_as_longlong(largest));
    }
    // The operands of the member sums below: this wavefront has 16 dimensions of 64 points, and their six digits or a share of
    // them.
    constexpr int GROUPS = NW / (2 * DT), DIGITS = (6 + GROUPS - 1) / GROUPS;   // wavefronts that share out the digits; of each
    const int sum_dt = wave % DT, sum_half = wave / DT % 2, sum_group = wave / (2 * DT);
    const bool sums_here = B.mt > 0 && 64 * sum_half < N && sum_group * DIGITS < 6;
    int4_t digits[DIGITS];
#pragma unroll
    for (int w = 0; w < 4; ++w) {   // four points each
        if (!sums_here) break;   // the same in every lane
        unsigned lo[4], hi[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int pt = 64 * sum_half + 16 * quarter + 4 * w + e;
            const float z = pt < 16 * PT ? Z[pt * zs + 16 * sum_dt + col] : 0.f;
            // 2^-32 fixed point plus 128 in every byte (coordinates beyond 2^13 take the other way below)
            const long long x = __double2ll_rn((double)z * 4294967296.0) + 0x808080808080ll;
            lo[e] = (unsigned)x, hi[e] = (unsigned)((unsigned long long)x >> 32);
        }
        // four words of four bytes -> the words of their lowest, second, ... bytes
        const unsigned a01 = __builtin_amdgcn_perm(lo[1], lo[0], 0x05010400u), a23 = __builtin_amdgcn_perm(lo[3], lo[2], 0x05010400u),
                       b01 = __builtin_amdgcn_perm(lo[1], lo[0], 0x07030602u), b23 = __builtin_amdgcn_perm(lo[3], lo[2], 0x07030602u),
                       c01 = __builtin_amdgcn_perm(hi[1], hi[0], 0x05010400u), c23 = __builtin_amdgcn_perm(hi[3], hi[2], 0x05010400u);
        const unsigned all[6] = {__builtin_amdgcn_perm(a23, a01, 0x05040100u), __builtin_amdgcn_perm(a23, a01, 0x07060302u),
                                 __builtin_amdgcn_perm(b23, b01, 0x05040100u), __builtin_amdgcn_perm(b23, b01, 0x07060302u),
                                 __builtin_amdgcn_perm(c23, c01, 0x05040100u), __builtin_amdgcn_perm(c23, c01, 0x07060302u)};
#pragma unroll
        for (int i = 0; i < DIGITS; ++i) {
            unsigned v = all[i];
#pragma unroll
            for (int g = 1; g < GROUPS; ++g)
                if (g * DIGITS + i < 6) v = sum_group == g ? all[g * DIGITS + i] : v;
            digits[i][w] = (int)(v ^ 0x80808080u);   // the byte less 128
        }
    }
    __syncthreads();
    // Bound on |score - exact score|, the score of a point z and a centroid c being |c - s|^2 - 2 (z - s).(c - s) about the middle
    // s.  With M = the largest |z - s|^2: a mean is formed from coordinates rounded to 2^-32, so it may lie up to 2^-33 per
    // coordinate outside the points' hull, and |c - s| is at most r = sqrt(M) + sqrt(d) 2^-33, r^2 at most 1.01 M + 101 d 2^-66
    // (plus its rounding to single precision, small against M unless s is 2^15 sqrt(M) away).  The differences' rounding makes
    // 7 u r^2 (u = 2^-24); |c - s|^2 takes 4 DT + 2 roundings of at most r^2, each of the two chains of products 8 DT + 2 sums
    // and their sum one more, of at most 3 r^2, the products 2 r^2 together; adding 2 delta to the smallest score below is one
    // more of 3 r^2: (28 DT + 23) u r^2, and one to spare; the rule's own error is far below.  What is closer than that goes to
    // the rule, one decision in some thousand, or all where the points lie closer together than the 2^-32.
    // (Double precision would be half the instructions' rate and twice the registers; without the middle, pairs far from the
    // origin would have all their points decided by the rule.)
    // With a coordinate that is not finite, or so large (2^24) that the 64-bit sum of 128 of them may wrap and leave
    // the hull, a middle that far away, or squares near single precision's smallest numbers there is no such bound: every
    // centroid is a candidate and the rule decides by itself.
    const double most_sq = __longlong_as_double(*(const long long *)(flags + 4));
    const double reach_sq = 1.01 * most_sq + 101.0 * (16 * DT) * 0x1p-66;
    const float two_delta = flags[6] || !(most_sq > 0x1p-80) || !((double)mid_sq < 0x1p30 * most_sq)
                                ? INFINITY
                                : (float)(2.0 * 1.01 * (double)(28 * DT + 24) * 0x1p-24 * reach_sq);
    const bool large = flags[3] != 0;
    const int tiles = B.mt * DT;
    const int iters = T_l > T_b ? T_l : T_b;   // 0 for what does not run
    // The bucket rule (fp64, dimensions in order, multiply and add separately, lowest index among equals) on
    // the candidates of the points that have several: `mine` has bit v set if centroid 4 v + quarter of run q
    // is a candidate of point pt (bits of rows that hold no centroid count for nothing); returns the winner's bit
    // alone, in the winner's lane.
    auto exact_winner = [&](unsigned mine, int pt, int q, int k) -> unsigned {
        unsigned cand = 0;
        for (int v = 0; v < 4; ++v) cand |= (mine >> v & 1u) << (4 * v + quarter);
        cand = quarter_or(cand) & ((1u << k) - 1u);
        int c = __builtin_ctz(cand);
        if (cand & (cand - 1)) {
            double best = 0.0;
            for (unsigned left = cand; left; left &= left - 1) {
                const int cc = __builtin_ctz(left);
                double D = 0.0;
                for (int j = 0; j < d; ++j) {
                    const double t = (double)Z[pt * zs + j] - (double)cent[(row_of(q) + cc) * zs + j];
                    const double t2 = t * t;
                    D = D + t2;
                }
                if (left == cand || D < best) {   // a first distance that is not a number keeps the point
                    best = D;
                    c = cc;
                }
            }
        }
        return (c & 3) == quarter ? 1u << (c >> 2) : 0u;
    };
    // Row i of a tile's operand holds centroid 4 (i % 4) + i / 4, so that lane l receives the scores of centroids
    // 4 v + l / 16: a run's are the same v in every lane.
    const int crow = 4 * (col & 3) + (col >> 2);
    unsigned valid = 0;   // bit t: row crow of centroid tile t holds a centroid
    for (int t = 0; t < B.mt; ++t) valid |= (start[16 * t + crow] >= 0 ? 1u : 0u) << t;
    unsigned held[TPW];   // by run, four bits: which of this lane's centroids had the point in the last iteration
#pragma unroll
    for (int u = 0; u < TPW; ++u) held[u] = 0u;
    for (int it = 0; it < iters && runs > 0; ++it) {
        int *cnt = cnts + (it & 1) * rows16;
        unsigned changed = 0;
        for (int mt = 0; mt < B.mt; ++mt) {
            // this tile's centroids as operands: -2 c, and one step more that adds |c|^2 (rows without a
            // centroid: a score no minimum picks)
            float aop[4 * DT], cn = 0.f;
#pragma unroll
            for (int t = 0; t < DT; ++t) {
                const float4 v = *(const float4 *)(cent + (16 * mt + crow) * zs + 16 * t + 4 * quarter);
                const float4 s = *(const float4 *)(mid + 16 * t + 4 * quarter);
                const float f[4] = {v.x - s.x, v.y - s.y, v.z - s.z, v.w - s.w};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    aop[4 * t + e] = -2.f * f[e];
                    cn = fmaf(f[e], f[e], cn);
                }
            }
            cn = quarter_sum(cn);
            const float an = quarter == 0 ? (valid >> mt & 1u ? cn : 1e38f) : 0.f;
            const float bn = quarter == 0 ? 1.f : 0.f;
#pragma unroll
            for (int u = 0; u < TPW; ++u) {
                const int tile = wave + NW * u;
                if (tile >= PT) continue;   // the same in every lane
                float4_t acc = {0.f, 0.f, 0.f, 0.f}, acc2 = {0.f, 0.f, 0.f, 0.f};   // two chains
                acc = __builtin_amdgcn_mfma_f32_16x16x4f32(an, bn, acc, 0, 0, 0);
#pragma unroll
                for (int e = 0; e < 4 * DT; e += 2) {
                    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(aop[e], zop[u][e], acc, 0, 0, 0);
                    acc2 = __builtin_amdgcn_mfma_f32_16x16x4f32(aop[e + 1], zop[u][e + 1], acc2, 0, 0, 0);
                }
                acc += acc2;
                const int pt = 16 * tile + col;
                for (int q = 0; q < runs; ++q) {
                    if (row_of(q) >> 4 != mt || it >= iters_of(q)) continue;   // the same in every lane
                    const int k = k_of(q), va = (row_of(q) & 15) >> 2, vb = va + ((k + 3) >> 2);
                    float best = INFINITY;
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        best = v >= va && v < vb ? min32(best, acc[v]) : best;
                    const float most = quarter_min(best) + two_delta;
                    // the lanes that hold a candidate; a column (point) in which two do is undecided
                    unsigned mine = 0;
                    unsigned long long seen = 0, twice = 0;
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                    {
                        // (not "at most": a score that is not a number is one the rule has to decide)
                        const bool in = v >= va && v < vb && !(acc[v] > most);
                        const unsigned long long b = __ballot(in);
                        mine |= in ? 1u << v : 0u;
                        twice |= seen & b;
                        seen |= b;
                    }
                    mine >>= va;
                    unsigned long long half = seen | seen >> 32;
                    twice |= (seen & seen >> 32) | (half & half >> 16);
                    if ((unsigned)(twice >> 32) | (unsigned)twice) mine = exact_winner(mine, pt, q, k);
                    const int shift = 4 * q;
                    const unsigned differs = (held[u] ^ mine << shift) & 15u << shift;
                    changed |= differs;
                    held[u] ^= differs;
                    if (mine && pt < N) {   // one lane per point
                        const int c = 4 * __builtin_ctz(mine) + quarter;
                        assign[q * L.rows + pt] = (unsigned char)c;
                        atomicAdd(&cnt[row_of(q) + c], 1);
                    }
                }
            }
        }
        if (__any(changed != 0) && lane == 0) flags[it & 1] = 1;
        __syncthreads();
        if (!flags[it & 1]) break;   // the same in every thread
        if (!large) {
            // Member sums in 2^-32 fixed point as products on the 8-bit matrix instruction, rows = centroids,
            // columns = dimensions, 64 points per instruction: of the 0/1 membership matrix with each of the six signed
            // digits to the base 256 (kept in registers) that a coordinate below 2^13 has, put together in double
            // precision: whole numbers below 2^52, exact in any order.
            if (sums_here)
                for (int mt = 0; mt < B.mt; ++mt) {
                    // the run and index of this lane's centroid row
                    const int own = owner[16 * mt + col];
                    const unsigned mine = own >= 0 ? (unsigned)(own & 255) * 0x01010101u : 0u;
                    const uint4 as = *(const uint4 *)(assign + (own >= 0 ? own >> 8 : 0) * L.rows + 64 * sum_half + 16 * quarter);
                    const unsigned a[4] = {as.x, as.y, as.z, as.w};
                    int4_t member;   // (both bytes are below 16, so nothing is borrowed from the next one)
#pragma unroll
                    for (int w = 0; w < 4; ++w)
                        member[w] = (int)((0x10101010u - ((a[w] ^ mine) & 0x0F0F0F0Fu)) >> 4 & 0x01010101u);
                    int4_t acc[DIGITS];
#pragma unroll
                    for (int i = 0; i < DIGITS; ++i)
                        acc[i] = __builtin_amdgcn_mfma_i32_16x16x64_i8(member, digits[i], int4_t{0, 0, 0, 0}, 0, 0, 0);
                    const double unit = ldexp(1.0, 8 * DIGITS * sum_group);
#pragma unroll
                    for (int v = 0; v < 4; ++v) {   // lane l has rows 4 (l / 16) + v
                        // three digits make a whole number below 2^30
                        int three[(DIGITS + 2) / 3] = {};
#pragma unroll
                        for (int i = 0; i < DIGITS; ++i) three[i / 3] += acc[i][v] << 8 * (i % 3);
                        double t = (double)three[0];
                        if constexpr (DIGITS > 3) t = fma((double)three[1], 0x1p24, t);
                        unsafeAtomicAdd(&sums[256 * (mt * DT + sum_dt) + 16 * (4 * quarter + v) + col], t * unit);
                    }
                }
        } else {
            // coordinates up to 2^31: 64-bit integers
            unsigned long long *isum = (unsigned long long *)sums;
            for (int e = tid; e < tiles * 256; e += NT) isum[e] = 0ull;
            __syncthreads();
            for (int e = tid; e < N * 16 * DT; e += NT) {
                const int i = e / (16 * DT), j = e % (16 * DT);
                const unsigned long long fx = (unsigned long long)__double2ll_rn((double)Z[i * zs + j] * 4294967296.0);
                for (int q = 0; q < runs; ++q) {
                    if (it >= iters_of(q)) continue;
                    const int row = row_of(q) + assign[q * L.rows + i];
                    atomicAdd(&isum[256 * ((row >> 4) * DT + (j >> 4)) + 16 * (row & 15) + (j & 15)], fx);
                }
            }
        }
        __syncthreads();
        for (int e = tid; e < 16 * DT * rows16; e += NT) {
            const int row = e / (16 * DT), j = e % (16 * DT);
            const int k = cnt[row], at = 256 * ((row >> 4) * DT + (j >> 4)) + 16 * (row & 15) + (j & 15);
            if (it < (row < landmark_rows ? T_l : T_b) && k > 0) {   // an empty cluster keeps its centroid
                const double sum = large ? (double)(long long)((const unsigned long long *)sums)[at] : sums[at];
                cent[row * zs + j] = (float)((sum * (1.0 / 4294967296.0)) / (double)k);
            }
            sums[at] = 0.0;   // for the next iteration
        }
        for (int e = tid; e < rows16; e += NT) cnts[((it + 1) & 1) * rows16 + e] = 0;
        if (tid == 0) flags[(it + 1) & 1] = 0;
        __syncthreads();
    }
    __syncthreads();   // a loop left early has its assignments in place, but other wavefronts may still read the flag

    constexpr int dp = 16 * DT;
    const double inv_lam = 1.0 / lam;
    // sixteen rows of Z or cent as a matrix operand of this lane
    auto operand = [&](const float *rows, int at, double (&o)[4 * DT]) {
#pragma unroll
        for (int t = 0; t < DT; ++t) {
            const float4 v = *(const float4 *)(rows + at * zs + 16 * t + 4 * quarter);
            o[4 * t] = (double)v.x, o[4 * t + 1] = (double)v.y, o[4 * t + 2] = (double)v.z, o[4 * t + 3] = (double)v.w;
        }
    };
    auto dots = [&](const double (&a)[4 * DT], const double (&b)[4 * DT]) -> double4_t {
        double4_t x = {0.0, 0.0, 0.0, 0.0}, y = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int e = 0; e < 4 * DT; e += 2) {
            x = __builtin_amdgcn_mfma_f64_16x16x4f64(a[e], b[e], x, 0, 0, 0);
            y = __builtin_amdgcn_mfma_f64_16x16x4f64(a[e + 1], b[e + 1], y, 0, 0, 0);
        }
        return x + y;
    };
    if (low_rank) {
        for (int e = tid; e < l * d; e += NT) B.landmarks[(long long)p * l * d + e] = cent[(e / d) * zs + e % d];
        // exp(-c / lambda) of the landmarks (rows 0 .. l - 1 of the first tile) with every point and among themselves.
        // Squared distances from the differences, not from dot products: what A^{-1} does to an error of these costs is
        // its condition number (two dimensions, sixteen landmarks, points 70 from the origin: K~ off by up to 5e-4
        // of itself from dot products, below its rounding to single precision from differences).
        const bool cosine = B.cost == LCN_COST_COSINE;
        double lop[4 * DT];
        if (cosine) {
            operand(cent, col, lop);
            double sq = 0.0;
#pragma unroll
            for (int e = 0; e < 4 * DT; ++e) sq = fma(lop[e], lop[e], sq);
            sq = quarter_sum(sq);
            if (wave == 0 && quarter == 0) rn[col] = sq;
            __syncthreads();   // the same in every thread
        }
        for (int t = wave; t <= PT; t += NW) {   // tile PT: the landmarks themselves
            const bool self = t == PT;
            const int pt = self ? col : 16 * t + col;
            const float *other = self ? cent : Z;
            double c[4] = {0.0, 0.0, 0.0, 0.0};   // of landmark 4 v + quarter and point pt
            if (cosine) {
                double bop[4 * DT];
                operand(other, pt, bop);
                const double4_t dot = dots(lop, bop);
                const double b2 = self ? rn[col] : pn[pt];
#pragma unroll
                for (int v = 0; v < 4; ++v) c[v] = 1.0 - dot[v] / (sqrt(rn[4 * v + quarter]) * sqrt(b2));
            } else {
#pragma unroll 4
                for (int k = 0; k < dp; k += 4) {
                    const float4 z = *(const float4 *)(other + pt * zs + k);
                    const double zd[4] = {(double)z.x, (double)z.y, (double)z.z, (double)z.w};
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        if (4 * v < l) {   // the same in every lane
                            const float4 f = *(const float4 *)(cent + (4 * v + quarter) * zs + k);
                            const double fd[4] = {(double)f.x, (double)f.y, (double)f.z, (double)f.w};
#pragma unroll
                            for (int e = 0; e < 4; ++e) {
                                const double diff = zd[e] - fd[e];
                                c[v] = fma(diff, diff, c[v]);
                            }
                        }
                }
                if (B.cost == LCN_COST_EUCLID) {
#pragma unroll
                    for (int v = 0; v < 4; ++v) c[v] = sqrt(c[v]);
                }
            }
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int k = 4 * v + quarter;
                if (k < l && pt < (self ? l : N)) {
                    const double f = exp(-(self && k == pt ? 0.0 : c[v]) * inv_lam);
                    if (self)
                        Am[k * l + pt] = f + (k == pt ? B.ridge : 0.0);
                    else
                        F[pt * L.ls + k] = f;
                }
            }
        }
        __syncthreads();
        const double *rdiag = Am + l * l;   // 1 / L_jj
        if (wave == 0) {
            if (l <= 8)
                landmark_cholesky<8>(Am, l, flags + 2);
            else
                landmark_cholesky<BL>(Am, l, flags + 2);
        }
        __syncthreads();
        // every point's factor row f -> L^{-1} f, a thread per point
        for (int i = tid; i < N; i += NT) {
            double *f = F + i * L.ls;
            double x[BL];
#pragma unroll
            for (int k = 0; k < BL; ++k) {
                if (k < l) {
                    double t = f[k];
#pragma unroll
                    for (int q = 0; q < k; ++q) t = fma(-Am[k * l + q], x[q], t);
                    x[k] = t * rdiag[k];
                    f[k] = x[k];
                }
            }
        }
        __syncthreads();
    }
    if (hashed)
        for (int r = 0; r < B.R; ++r)
            for (int i = tid; i < N; i += NT)
                B.buckets[(x0 + y0) * B.R + (long long)r * N + i] = assign[(first_hash + r) * L.rows + i];
    // K~_ij: exact where x_i and y_j share a bucket, Nystrom elsewhere (0 without a Nystrom part); a
    // wavefront takes 16 x 16 tiles, rows x_i, columns y_j
    float *Kt = B.Kt + (long long)p * BMAX * BMAX;
    const int TI = (n + 15) / 16, TJ = (m + 15) / 16;
    // A quarter of a pair's entries or so are near, spread over all lanes: they are put into a list and taken from it 64 at a
    // time, so that costs and exponentials are formed for full wavefronts (4096 pairs: the build's call 303 -> 297 us, 1024: 115 -> 111).
    NearList &near_list = ((NearList *)cent)[wave];
    int listed = 0, done = 0;   // entries put in and taken out so far
    auto form = [&](int count) {   // the next `count` entries, up to 64
        __builtin_amdgcn_wave_barrier();
        if (lane < count) {
            const int at = (done + lane) & 127, place = near_list.place[at], i = place >> 6, j = place & 63;
            const double c = cost_of_dot(near_list.dot[at], pn[i], pn[n + j], Z + i * zs, Z + (n + j) * zs, dp, B.cost);
            Kt[place] = (float)exp(-c * inv_lam);
        }
        done += count;
        __builtin_amdgcn_wave_barrier();
    };
    static_assert(BMAX == 64, "place of a kernel entry");
    for (int t = wave; t < TI * TJ; t += NW) {
        const int ti = t / TJ, tj = t % TJ;
        const int j = 16 * tj + col;
        const int ar = 16 * ti + col < n ? 16 * ti + col : n - 1, br = n + (j < m ? j : m - 1);   // operand rows
        bool near[4];
        bool any_near = false;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int i = 16 * ti + 4 * v + quarter;
            const bool in = i < n && j < m;
            near[v] = in && B.mode == LCN_MODE_DENSE;
#pragma unroll
            for (int r = 0; r < BR; ++r)
                if (r < B.R) {
                    const unsigned char *as = assign + (first_hash + r) * L.rows;
                    near[v] = near[v] || (in && as[i < n ? i : n - 1] == as[br]);
                }
            any_near = any_near || near[v];
        }
        double4_t nys = {0.0, 0.0, 0.0, 0.0}, dot = {0.0, 0.0, 0.0, 0.0};
        if (low_rank) {
            for (int k = quarter; k - quarter < l; k += 4)
                nys = __builtin_amdgcn_mfma_f64_16x16x4f64(k < l ? F[ar * L.ls + k] : 0.0,
                                                          k < l ? F[br * L.ls + k] : 0.0, nys, 0, 0, 0);
        }
        if (__any(any_near)) {
            double xop[4 * DT], yop[4 * DT];
            operand(Z, ar, xop);
            operand(Z, br, yop);
            dot = dots(xop, yop);
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int place = (16 * ti + 4 * v + quarter) * BMAX + j;
            const unsigned long long here = __ballot(near[v]);
            if (near[v]) {
                const int at = (listed + __builtin_amdgcn_mbcnt_hi((unsigned)(here >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)here, 0u))) & 127;
                near_list.dot[at] = dot[v];
                near_list.place[at] = (unsigned short)place;
            } else if (16 * ti + 4 * v + quarter < n && j < m) {
                Kt[place] = (float)nys[v];
            }
            listed += __popcll(here);
            if (listed - done >= 64) form(64);
        }
    }
    form(listed - done);
    if (B.bp) {
        for (int i = tid; i < n; i += NT) B.kpe[x0 + i] = exp(-(double)B.del_x[x0 + i] / lam);
        for (int i = tid; i < m; i += NT) B.keq[y0 + i] = exp(-(double)B.del_y[y0 + i] / lam);
    }
    const int len_u = B.bp ? N : n, len_v = B.bp ? N : m;
    for (int i = tid; i < len_u; i += NT) B.log_u[x0 + y0 + i] = 0.0;
    for (int i = tid; i < len_v; i += NT) B.log_v[x0 + y0 + i] = 0.0;
    if (tid == 0 && flags[2]) B.marks[0] = 1;
}

constexpr int RUN_PAIRS = 4;   // of a workgroup of the run kernel at most, one per SIMD of a compute unit

// iters Sinkhorn iterations per pair (iters == 0: only the query part), then the
// pair's distance and marginal residual.
//
// One wavefront per pair, no workgroup-wide step and no LDS anywhere.  The pair's 64 x 64 kernel tile
// (zero beyond n x m) is dealt to the lanes in 8 x 8 blocks, held as doubles: lane (r, c) = 8 r + c owns
// rows 8 r .. 8 r + 7 and columns 8 c .. 8 c + 7, ONE copy that serves both products.  A product is 64
// multiply-adds on registers and a sum over the eight lanes that share the rows (columns), done by
// recursive halving, 4 + 2 + 1 exchanges: afterwards every lane holds ONE row (column) of the result,
// row 8 r + c (column 8 c + r), scales it, and the next product's eight inputs come back by recursive
// doubling.  Which of a block's rows a register holds depends on the lane (row 8 r + (sigma(k) ^ c) in
// register k, sigma the masks of the three lane permutations), so the halving needs no selects; along
// the columns two of the three exchanges are lane swaps, which select by themselves.
// What bounds it is one wavefront's instruction stream: about 170 vector instructions per
// half-iteration, 64 of them the product itself (the version before it, a row and a column per lane with
// the vector passed round by lane reads, needed 330).  50 iterations of 4096 pairs with deletion rows:
// 157 us, of 16 pairs 47.
//
// The entries of u = [u^ (n); u~ (m)] and v = [v^ (m); v~ (n)] (point part; deletion part, Sec. 6) live
// where the products leave them: u^_i and v~_i in the lane of row i, v^_j and u~_j in the lane of column j.
// A vector is held as x * 2^E with one integer E for the whole vector, the largest entry kept within
// 2^-40 .. 2^40: the max-shift of App. "Implementational details" with the shift restricted to powers
// of two and applied when it is due, which costs two comparisons per half-iteration instead of an exp
// and a log per entry.  Logs are formed once, when the state is stored.
//   (K_BP v)_i     = sum_j K_ij v^_j + k_{i,eps} v~_i          (K_BP v)_{n+j}     = k_{eps,j} v^_j + sum v~
//   (K_BP^T u)_j   = sum_i K_ij u^_i + k_{eps,j} u~_j          (K_BP^T u)_{m+i}   = k_{i,eps} u^_i + sum u~
template <bool BP>
__global__ __launch_bounds__(64 * RUN_PAIRS, 2) void batched_run_kernel(BatchDev B, int iters, float *row_marg, float *col_marg)
{
    const double LN2 = 0.69314718055994530942;
    const int p = (int)(blockIdx.x * (blockDim.x >> 6)) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (p >= B.P) return;
    const long long x0 = B.x_off[p], y0 = B.y_off[p];
    const int n = (int)(B.x_off[p + 1] - x0), m = (int)(B.y_off[p + 1] - y0);
    const int len_u = BP ? n + m : n, len_v = BP ? n + m : m;
    const int lr = lane >> 3, lc = lane & 7;
    const int row = lane, col = 8 * lc + lr;   // this lane's entry of a result over rows / over columns
    // the lane permutations of the row sums: xor 7 (half mirror), xor 2, xor 1
    constexpr int SIG[8] = {0, 1, 2, 3, 7, 6, 5, 4};
    double K[8][8];
    {
        const float *Kt = B.Kt + (long long)p * BMAX * BMAX;
        float4 raw[8][2];
#pragma unroll
        for (int a = 0; a < 8; ++a) {
            const int i = 8 * lr + (SIG[a] ^ lc);
#pragma unroll
            for (int q = 0; q < 2; ++q)   // the tile is stored 64 x 64 whatever n and m: always readable
                raw[a][q] = *(const float4 *)(Kt + i * BMAX + 8 * lc + 4 * q);
        }
        // columns 2 g and 2 g + 1 trade places in the odd rows of lanes
        const bool odd = lr & 1;
        const int j_even = 8 * lc + (odd ? 1 : 0), j_odd = 8 * lc + (odd ? 0 : 1);
#pragma unroll
        for (int a = 0; a < 8; ++a) {
            const bool in_row = 8 * lr + (SIG[a] ^ lc) < n;
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                float f0 = odd ? raw[a][q].y : raw[a][q].x, f1 = odd ? raw[a][q].x : raw[a][q].y;
                float f2 = odd ? raw[a][q].w : raw[a][q].z, f3 = odd ? raw[a][q].z : raw[a][q].w;
                f0 = in_row && j_even + 4 * q < m ? f0 : 0.f;
                f1 = in_row && j_odd + 4 * q < m ? f1 : 0.f;
                f2 = in_row && j_even + 4 * q + 2 < m ? f2 : 0.f;
                f3 = in_row && j_odd + 4 * q + 2 < m ? f3 : 0.f;
                K[a][4 * q] = (double)f0;
                K[a][4 * q + 1] = (double)f1;
                K[a][4 * q + 2] = (double)f2;
                K[a][4 * q + 3] = (double)f3;
            }
        }
    }
    const bool has_up = row < n, has_ud = BP && col < m;   // this lane's entries of u (point, deletion part)
    const bool has_vp = col < m, has_vd = BP && row < n;   // ... and of v
    const double kpe = has_vd ? B.kpe[x0 + row] : 0.0;
    const double keq = has_ud ? B.keq[y0 + col] : 0.0;
    double *gu = B.log_u + x0 + y0, *gv = B.log_v + x0 + y0;
    const double a_each = 1.0 / (double)len_u, b_each = 1.0 / (double)len_v;   // uniform marginals
    unsigned long long nonpos = 0, empty_u = 0, empty_v = 0;
    // A kernel without a Nystrom part and without deletion entries has no signed terms: a sum of
    // exactly zero means the point shares no bucket with any point of the other set (or only
    // vanished entries).  Such a point gets scaling 0 (log = -infinity), carries no mass and is
    // counted apart from the non-positive sums (App. "Limitations": ignored, not a failure).
    const bool unsupported_is_zero = !BP && B.l == 0;

    // stored logs -> x * 2^E
    auto load_vec = [&](double lp, bool hp, double ld, bool hd, double &xp, double &xd) -> int {
        const double M = wave_max(fmax(hp ? lp : -INFINITY, hd ? ld : -INFINITY));
        const double Ms = (M > -INFINITY && M < INFINITY) ? M : 0.0;
        const double Ef = floor(Ms * 1.4426950408889634074);
        xp = hp ? exp(lp - Ef * LN2) : 0.0;
        xd = hd ? exp(ld - Ef * LN2) : 0.0;
        return (int)Ef;
    };
    // Once the largest entry has left 2^-40 .. 2^40: back into [1, 2); returns the exponent taken out
    // (NaN entries are ignored by the comparisons and by fmax)
    auto renorm = [&](double &xp, double &xd) -> int {
        const double own = fmax(xp, xd);
        if (!__any(own > 0x1p40) && __any(own > 0x1p-40)) return 0;
        const double mx = wave_max(own);
        if (!(mx > 0.0) || !(mx < INFINITY)) return 0;
        const int e = ilogb(mx);
        xp = ldexp(xp, -e);
        xd = ldexp(xd, -e);
        return e;
    };
    // s_row = this lane's row of K times the vector whose entries (one per lane, by column) are x
    auto times_rows = [&](double x) -> double {
        double in[8], acc[8];
        in[0] = x;
        in[1] = dpp_from<0x128>(in[0]);   // row_ror:8
#pragma unroll
        for (int g = 0; g < 2; ++g) {
            in[g + 2] = in[g];
            lane_swap<16>(in[g], in[g + 2]);
        }
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            in[g + 4] = in[g];
            lane_swap<32>(in[g], in[g + 4]);
        }
#pragma unroll
        for (int a = 0; a < 8; ++a) acc[a] = K[a][0] * in[0];
#pragma unroll
        for (int b = 1; b < 8; ++b)
#pragma unroll
            for (int a = 0; a < 8; ++a) acc[a] = fma(K[a][b], in[b], acc[a]);
#pragma unroll
        for (int a = 0; a < 4; ++a) acc[a] += dpp_from<0x141>(acc[a + 4]);   // row_half_mirror
#pragma unroll
        for (int a = 0; a < 2; ++a) acc[a] += dpp_from<0x4E>(acc[a + 2]);    // xor 2
        return acc[0] + dpp_from<0xB1>(acc[1]);                              // xor 1
    };
    // s_col = this lane's column of K times the vector whose entries (one per lane, by row) are x
    auto times_cols = [&](double x) -> double {
        double in[8], acc[8];
        in[0] = x;
        in[1] = dpp_from<0xB1>(in[0]);
#pragma unroll
        for (int a = 0; a < 2; ++a) in[a + 2] = dpp_from<0x4E>(in[a]);
#pragma unroll
        for (int a = 0; a < 4; ++a) in[a + 4] = dpp_from<0x141>(in[a]);
#pragma unroll
        for (int b = 0; b < 8; ++b) acc[b] = K[0][b] * in[0];
#pragma unroll
        for (int a = 1; a < 8; ++a)
#pragma unroll
            for (int b = 0; b < 8; ++b) acc[b] = fma(K[a][b], in[a], acc[b]);
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            lane_swap<32>(acc[b], acc[b + 4]);
            acc[b] += acc[b + 4];
        }
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            lane_swap<16>(acc[b], acc[b + 2]);
            acc[b] += acc[b + 2];
        }
        return acc[0] + dpp_from<0x128>(acc[1]);
    };
    auto scale = [&](double marg, double s, bool exists, unsigned long long &empty) -> double {
        if (!exists) return 0.0;
        if (s > 0.0) return marg * fast_rcp(s);
        if (unsupported_is_zero && s == 0.0) {
            ++empty;
            return 0.0;
        }
        ++nonpos;
        return NAN;
    };
    // sums of K_BP v: of this lane's row, and of its column's deletion row; and the same of K_BP^T u
    auto rows_of = [&](double vp, double vd, double &s_p, double &s_d) {
        const double tail = BP ? wave_sum(vd) : 0.0;
        s_p = times_rows(vp);
        if (BP) s_p = fma(kpe, vd, s_p);
        s_d = fma(keq, vp, tail);
    };
    auto cols_of = [&](double up, double ud, double &s_p, double &s_d) {
        const double tail = BP ? wave_sum(ud) : 0.0;
        s_p = times_cols(up);
        if (BP) s_p = fma(keq, ud, s_p);
        s_d = fma(kpe, up, tail);
    };

    double xu_p = 0.0, xu_d = 0.0, xv_p, xv_d, s_p, s_d;
    int Eu = 0;
    int Ev = load_vec(has_vp ? gv[col] : 0.0, has_vp, has_vd ? gv[m + row] : 0.0, has_vd, xv_p, xv_d);
    if (iters == 0) Eu = load_vec(has_up ? gu[row] : 0.0, has_up, has_ud ? gu[n + col] : 0.0, has_ud, xu_p, xu_d);
    for (int it = 0; it < iters; ++it) {
        rows_of(xv_p, xv_d, s_p, s_d);        // u = a ./ (K_BP v), eq. 2
        xu_p = scale(a_each, s_p, has_up, empty_u);
        if (BP) xu_d = scale(a_each, s_d, has_ud, empty_u);
        Eu = -Ev + renorm(xu_p, xu_d);
        cols_of(xu_p, xu_d, s_p, s_d);        // v = b ./ (K_BP^T u)
        xv_p = scale(b_each, s_p, has_vp, empty_v);
        if (BP) xv_d = scale(b_each, s_d, has_vd, empty_v);
        Ev = -Eu + renorm(xv_p, xv_d);
    }
    const double lu_p = log(xu_p) + (double)Eu * LN2, lu_d = log(xu_d) + (double)Eu * LN2;
    const double lv_p = log(xv_p) + (double)Ev * LN2, lv_d = log(xv_d) + (double)Ev * LN2;
    if (iters > 0) {
        if (has_up) gu[row] = lu_p;
        if (has_ud) gu[n + col] = lu_d;
        if (has_vp) gv[col] = lv_p;
        if (has_vd) gv[m + row] = lv_d;
        nonpos = (unsigned long long)wave_sum((double)nonpos);
        empty_u = (unsigned long long)wave_sum((double)empty_u);
        empty_v = (unsigned long long)wave_sum((double)empty_v);
        if (lane == 0 && (nonpos | empty_u | empty_v)) B.marks[1] = 1;
        if (lane == 0 && nonpos) atomicAdd(&B.counters[0], nonpos);
        if (lane == 0 && empty_u) atomicAdd(&B.counters[1], empty_u);
        if (lane == 0 && empty_v) atomicAdd(&B.counters[2], empty_v);
    }

    // marginals r = u .* (K_BP v), c = v .* (K_BP^T u); distance and residual
    double dsum = 0.0, esum = 0.0;
    rows_of(xv_p, xv_d, s_p, s_d);
    if (has_up) {
        const double r = ldexp(xu_p * s_p, Eu + Ev);
        if (r != 0.0) dsum += r * lu_p;   // a point without mass (log u = -infinity) adds nothing
        esum += fabs(r - a_each);
        if (row_marg) row_marg[x0 + y0 + row] = (float)r;
    }
    if (has_ud) {
        const double r = ldexp(xu_d * s_d, Eu + Ev);
        dsum += r * lu_d;
        esum += fabs(r - a_each);
        if (row_marg) row_marg[x0 + y0 + n + col] = (float)r;
    }
    cols_of(xu_p, xu_d, s_p, s_d);
    if (has_vp) {
        const double c = ldexp(xv_p * s_p, Eu + Ev);
        if (c != 0.0) dsum += c * lv_p;
        esum += fabs(c - b_each);
        if (col_marg) col_marg[x0 + y0 + col] = (float)c;
    }
    if (has_vd) {
        const double c = ldexp(xv_d * s_d, Eu + Ev);
        dsum += c * lv_d;
        esum += fabs(c - b_each);
        if (col_marg) col_marg[x0 + y0 + m + row] = (float)c;
    }
    const double D = wave_sum(dsum);
    const double E = wave_sum(esum);
    if (lane == 0) {
        B.dist[p] = (double)B.lambda[p] * D;
        B.resid[p] = E;
    }
}

// c_i = || alpha .* x_i ||_2 (Sec. 6, learnable deletion cost); one thread per
// point, squares added in fp64 in the order of the dimensions.  The rows come through LDS, 32 dimensions of 256 points
// at a time in whole lines (a thread that reads its row by itself asks for 64 lines per load).
__global__ __launch_bounds__(256) void deletion_cost_kernel(const float *__restrict__ X, long long total, int d,
                                                            const float *__restrict__ alpha, float *__restrict__ out)
{
    __shared__ float rows[256][33];
    const long long i0 = (long long)blockIdx.x * 256;
    const int dim = threadIdx.x & 31, r0 = threadIdx.x >> 5;
    double s = 0.0;
    for (int k0 = 0; k0 < d; k0 += 32) {
        const int k = k0 + dim < d ? k0 + dim : d - 1;
        float v[32];
#pragma unroll
        for (int u = 0; u < 32; ++u) {   // past the last point or dimension: the last one again, not used
            const long long i = i0 + r0 + 8 * u < total ? i0 + r0 + 8 * u : total - 1;
            v[u] = X[i * d + k];
        }
        if (k0 > 0) __syncthreads();   // the dimensions before have been added
#pragma unroll
        for (int u = 0; u < 32; ++u) rows[r0 + 8 * u][dim] = v[u];
        __syncthreads();
        const int m = d - k0 < 32 ? d - k0 : 32;
#pragma unroll 8
        for (int e = 0; e < m; ++e) {
            const double t = (double)rows[threadIdx.x][e] * (double)alpha[k0 + e];
            s += t * t;
        }
    }
    if (i0 + threadIdx.x < total) out[i0 + threadIdx.x] = (float)sqrt(s);
}

// The batch's description into the workspace and the counters at zero, in one launch: from pinned host memory that the
// device reads itself.  words: multiples of 4 bytes.
__global__ __launch_bounds__(256) void batch_upload_kernel(const unsigned *__restrict__ src, unsigned *__restrict__ dst,
                                                           long long words, unsigned *counters, int counter_words)
{
    const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
    if (i < words) dst[i] = src[i];
    if (i < counter_words) counters[i] = 0u;
}

// The marginals of the last run to where the caller wants them (either may be null); a workgroup per pair, since the
// entries between the pairs are not the library's to write where there are no deletion entries.
__global__ __launch_bounds__(128) void batch_marginals_kernel(BatchDev B, float *__restrict__ rows, float *__restrict__ cols)
{
    const long long x0 = B.x_off[blockIdx.x], y0 = B.y_off[blockIdx.x];
    const int n = (int)(B.x_off[blockIdx.x + 1] - x0), m = (int)(B.y_off[blockIdx.x + 1] - y0);
    const int i = threadIdx.x;   // at most BMAX + BMAX entries
    if (rows && i < (B.bp ? n + m : n)) rows[x0 + y0 + i] = B.row_marg[x0 + y0 + i];
    if (cols && i < (B.bp ? n + m : m)) cols[x0 + y0 + i] = B.col_marg[x0 + y0 + i];
}

// What a batch handle needs of the host: a block of pinned memory that the kernels read the description from and
// write distances and marks to (a copy by the runtime costs more than these few bytes), and the events around a run.
// Made once and kept: at most HOST_BLOCKS idle ones and HOST_BYTES in all, the rest is given back at once.
struct HostBlock {
    int device;
    char *ptr;
    size_t bytes;
    hipEvent_t ev0, ev1;
};
constexpr size_t HOST_BLOCKS = 8, HOST_BYTES = (size_t)16 << 20;

// Room for them all from the start, so that nothing here allocates on the host, and nothing to do when the process ends: the
// runtime may be gone by then.
struct HostPool {
    std::mutex mu;
    size_t count;
    HostBlock idle[HOST_BLOCKS];
};
static_assert(std::is_trivially_destructible<HostPool>::value, "blocks are not given back at the end of the process");
static HostPool host_pool;

static void free_host_block(HostBlock &b)
{
    if (b.ev0) (void)hipEventDestroy(b.ev0);
    if (b.ev1) (void)hipEventDestroy(b.ev1);
    if (b.ptr) (void)hipHostFree(b.ptr);
    b = HostBlock{};
}

static hipError_t take_host_block(size_t bytes, HostBlock &out)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    {
        HostPool &pool = host_pool;
        std::lock_guard<std::mutex> lock(pool.mu);
        size_t best = pool.count;
        for (size_t i = 0; i < pool.count; ++i)
            if (pool.idle[i].device == dev && pool.idle[i].bytes >= bytes &&
                (best == pool.count || pool.idle[i].bytes < pool.idle[best].bytes))
                best = i;
        if (best < pool.count) {
            out = pool.idle[best];
            pool.idle[best] = pool.idle[--pool.count];
            return hipSuccess;
        }
    }
    HostBlock b{};
    b.device = dev;
    b.bytes = (size_t)1 << 16;
    while (b.bytes < bytes) b.bytes *= 2;
    e = hipHostMalloc((void **)&b.ptr, b.bytes, hipHostMallocDefault);
    if (e == hipSuccess) e = hipEventCreate(&b.ev0);
    if (e == hipSuccess) e = hipEventCreate(&b.ev1);
    if (e != hipSuccess) {
        free_host_block(b);
        return e;
    }
    out = b;
    return hipSuccess;
}

// (nothing on the device uses it any more)
static void give_host_block(HostBlock &b)
{
    if (!b.ptr) return;
    bool kept = false;
    {
        HostPool &pool = host_pool;
        std::lock_guard<std::mutex> lock(pool.mu);
        size_t held = b.bytes;
        for (size_t i = 0; i < pool.count; ++i) held += pool.idle[i].bytes;
        if (pool.count < HOST_BLOCKS && held <= HOST_BYTES) {
            pool.idle[pool.count++] = b;
            kept = true;
        }
    }
    if (kept)
        b = HostBlock{};
    else
        free_host_block(b);
}

struct BatchHandle {
    uint32_t magic;
    BatchDev dev;
    hipStream_t stream;
    long long total_x, total_y;
    size_t ws_used;
    HostBlock host;
    float last_ms;   // of the last run; < 0: still to be asked from its events
    bool run_done;   // dist, resid and the marginals are those of the present state
};

}  // namespace lcn

using namespace lcn;

#define BHIPCHK(expr)                 \
    do {                              \
        hipError_t e_ = (expr);       \
        if (e_ != hipSuccess) {       \
            (void)hipGetLastError();  \
            return LCN_ERR_DEVICE;    \
        }                             \
    } while (0)

namespace lcn {
bool is_batched_handle(const void *h) { return h && *(const uint32_t *)h == BATCH_MAGIC; }

template <int NT, int DT>
static hipError_t launch_batched_build_as(const BatchHandle &h)
{
    const BatchDev &D = h.dev;
    const size_t bytes = build_lds(D.l, (D.l > 0 ? 1 : 0) + D.R, D.mt, DT, D.max_points, NT / 64).bytes;
    if (bytes > 64 * 1024) {   // has to be allowed
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&batched_build_kernel<NT, DT>),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL((batched_build_kernel<NT, DT>), dim3(D.P), dim3(NT), bytes, h.stream, D);
    return hipGetLastError();
}

// Eight wavefronts instead of four per pair: where a compute unit has at most two pairs and the pairs more
// than the four tiles of points that four wavefronts hold (what a call takes less, d = 32, 16 to 64 points per
// side: 64 pairs 11 us, 512 pairs 9, 768 pairs -18, 1024 pairs -18; 10 to 30 points: 64 pairs 3, 512 pairs 2, 768 pairs -13), and for more
// than 32 dimensions, where four wavefronts have too few registers for their points (1024 pairs, d = 64: 42 us).
static hipError_t launch_batched_build(const BatchHandle &h)
{
    const BatchDev &D = h.dev;
    const int dt = (D.d + 15) / 16;
    const bool wide = D.P <= 2 * device_compute_units() && D.max_points > 64;
    if (dt <= 1) return wide ? launch_batched_build_as<512, 1>(h) : launch_batched_build_as<256, 1>(h);
    if (dt == 2) return wide ? launch_batched_build_as<512, 2>(h) : launch_batched_build_as<256, 2>(h);
    return launch_batched_build_as<512, 4>(h);
}

// Four pairs per workgroup are one per SIMD; left to the dispatcher one by one, which SIMDs get two of them depends on what ran
// before (1024 pairs, 50 iterations, after their build: 63 us, one by one 89).  Where every pair can have a compute unit, one by one
// (50 iterations without deletion entries 48.5 us instead of 50.7, with them 59.2 / 60.5).
// Nothing keeps two workgroups of a run apart: with half a compute unit's LDS reserved per workgroup for that, a run by itself took
// the same (1024 pairs: 63 us), two on two streams one after the other (400 iterations: 671 us instead of 500).
static hipError_t launch_batched_run(const BatchHandle &h, int iters, float *row_dev, float *col_dev)
{
    const int each = h.dev.P <= device_compute_units() ? 1 : RUN_PAIRS;
    const dim3 grid((h.dev.P + each - 1) / each), block(64 * each);
    if (h.dev.bp)
        hipLaunchKernelGGL(batched_run_kernel<true>, grid, block, 0, h.stream, h.dev, iters, row_dev, col_dev);
    else
        hipLaunchKernelGGL(batched_run_kernel<false>, grid, block, 0, h.stream, h.dev, iters, row_dev, col_dev);
    return hipGetLastError();
}

lcn_status batched_run(void *hh, int iters)
{
    BatchHandle &h = *(BatchHandle *)hh;
    BHIPCHK(hipEventRecord(h.host.ev0, h.stream));
    h.run_done = false;
    BHIPCHK(launch_batched_run(h, iters, h.dev.row_marg, h.dev.col_marg));
    BHIPCHK(hipEventRecord(h.host.ev1, h.stream));
    h.last_ms = -1.f;
    BHIPCHK(hipStreamSynchronize(h.stream));
    h.run_done = true;
    if (!*(volatile int *)(h.dev.marks + 1)) return LCN_OK;
    unsigned long long c[3] = {0, 0, 0};
    const lcn_status st = batched_counts(hh, c);
    if (st != LCN_OK) return st;
    if (c[0]) return LCN_ERR_NONPOSITIVE;
    return (c[1] | c[2]) ? LCN_WARN_NO_SUPPORT : LCN_OK;
}

lcn_status batched_query(void *hh, double *dist_host, double *resid_host, float *row_dev, float *col_dev)
{
    BatchHandle &h = *(BatchHandle *)hh;
    // A run leaves all of this; forming the marginals again means reading every kernel again (4096 pairs: 26 us against 6).
    if (h.run_done && h.dev.row_marg) {
        if (row_dev || col_dev) {
            hipLaunchKernelGGL(batch_marginals_kernel, dim3(h.dev.P), dim3(2 * BMAX), 0, h.stream, h.dev, row_dev, col_dev);
            BHIPCHK(hipGetLastError());
        }
    } else {
        BHIPCHK(launch_batched_run(h, 0, row_dev, col_dev));
    }
    BHIPCHK(hipStreamSynchronize(h.stream));
    if (dist_host) memcpy(dist_host, h.dev.dist, sizeof(double) * h.dev.P);
    if (resid_host) memcpy(resid_host, h.dev.resid, sizeof(double) * h.dev.P);
    return LCN_OK;
}

lcn_status batched_counts(void *hh, unsigned long long c[3])
{
    BatchHandle &h = *(BatchHandle *)hh;
    BHIPCHK(hipMemcpyAsync(c, h.dev.counters, 3 * sizeof(unsigned long long), hipMemcpyDeviceToHost, h.stream));
    BHIPCHK(hipStreamSynchronize(h.stream));
    return LCN_OK;
}

lcn_status batched_timing(void *hh, float *ms, int *launches)
{
    BatchHandle &h = *(BatchHandle *)hh;
    if (h.last_ms < 0.f) BHIPCHK(hipEventElapsedTime(&h.last_ms, h.host.ev0, h.host.ev1));
    if (ms) *ms = h.last_ms;
    if (launches) *launches = 1;
    return LCN_OK;
}

void batched_destroy(void *hh)
{
    BatchHandle *h = (BatchHandle *)hh;
    (void)hipStreamSynchronize(h->stream);
    give_host_block(h->host);
    h->magic = 0;
    delete h;
}
}  // namespace lcn

extern "C" {

lcn_status lcn_build_batched(const float *X, const float *Y, int32_t d, const lcn_batch_desc *desc, int32_t cost,
                             int32_t mode, const lcn_landmark_params *lm, const lcn_lsh_params *lsh, void *workspace,
                             size_t workspace_bytes, void *hip_stream, size_t *bytes_needed, lcn_handle *out)
{
    if (!out) return LCN_ERR_INVALID_ARG;
    *out = nullptr;
    if (!X || !Y || !desc || !desc->x_off || !desc->y_off || !desc->lambda || !workspace ||
        ((uintptr_t)workspace & 255))
        return LCN_ERR_INVALID_ARG;
    const int P = desc->num_problems;
    if (P < 1 || d < 1 || d > BD) return LCN_ERR_INVALID_ARG;
    if (cost < LCN_COST_SQEUCLID || cost > LCN_COST_COSINE || mode < LCN_MODE_DENSE || mode > LCN_MODE_LCN)
        return LCN_ERR_INVALID_ARG;
    const bool low_rank = mode == LCN_MODE_NYSTROM || mode == LCN_MODE_LCN;
    const bool hashed = mode == LCN_MODE_SPARSE || mode == LCN_MODE_LCN;
    if (low_rank && (!lm || lm->num_landmarks < 1 || lm->num_landmarks > BL || lm->kmeans_iters < 1 || lm->init != LCN_INIT_SAMPLE ||
                     !(lm->ridge >= 0.0)))
        return LCN_ERR_INVALID_ARG;
    if (hashed && (!lsh || lsh->hash != LCN_HASH_KMEANS || lsh->num_buckets < 1 || lsh->num_buckets > BL ||
                   lsh->num_rounds < 1 || lsh->num_rounds > BR || lsh->kmeans_iters < 1 || lsh->branching[0] != 0 ||
                   lsh->and_width > 1))
        return LCN_ERR_INVALID_ARG;
    if ((desc->del_cost_x == nullptr) != (desc->del_cost_y == nullptr)) return LCN_ERR_INVALID_ARG;
    int max_points = 0;
    for (int p = 0; p < P; ++p) {
        const long long n = desc->x_off[p + 1] - desc->x_off[p], m = desc->y_off[p + 1] - desc->y_off[p];
        if (n < 1 || m < 1 || n > BMAX || m > BMAX) return LCN_ERR_INVALID_ARG;
        max_points = n + m > max_points ? (int)(n + m) : max_points;
        if (low_rank && lm->num_landmarks > n + m) return LCN_ERR_INVALID_ARG;
        if (hashed && lsh->num_buckets > n + m) return LCN_ERR_INVALID_ARG;
        if (!(desc->lambda[p] > 0.f)) return LCN_ERR_INVALID_ARG;
    }
    if (desc->x_off[0] != 0 || desc->y_off[0] != 0) return LCN_ERR_INVALID_ARG;
    const long long tx = desc->x_off[P], ty = desc->y_off[P];

    BatchHandle *hp = new (std::nothrow) BatchHandle{};
    if (!hp) return LCN_ERR_ALLOC;
    BatchHandle &h = *hp;
    struct Guard {
        BatchHandle *p;
        ~Guard()
        {
            if (p) {
                if (p->host.ptr) (void)hipStreamSynchronize(p->stream);   // a kernel may still use it
                give_host_block(p->host);
                delete p;
            }
        }
    } guard{hp};
    h.stream = (hipStream_t)hip_stream;
    h.total_x = tx;
    h.total_y = ty;
    BatchDev &D = h.dev;
    D.P = P;
    D.d = d;
    D.max_points = max_points;
    D.cost = cost;
    D.mode = mode;
    D.l = low_rank ? lm->num_landmarks : 0;
    D.b = hashed ? lsh->num_buckets : 1;
    D.R = hashed ? lsh->num_rounds : 0;
    D.T_l = low_rank ? lm->kmeans_iters : 0;
    D.T_b = hashed ? lsh->kmeans_iters : 0;
    D.seed_l = low_rank ? lm->seed : 0;
    D.seed_b = hashed ? lsh->seed : 0;
    D.ridge = low_rank ? lm->ridge : 0.0;
    build_rows(D);
    D.bp = desc->del_cost_x ? 1 : 0;
    D.X = X;
    D.Y = Y;
    D.del_x = desc->del_cost_x;
    D.del_y = desc->del_cost_y;

    char *base = (char *)workspace;
    size_t used = 0;
    auto take = [&](size_t bytes) -> void * {
        bytes = (bytes + 255) & ~(size_t)255;
        void *ptr = base + used;
        used += bytes;
        return ptr;
    };
    long long *xo = (long long *)take(sizeof(long long) * (P + 1));
    long long *yo = (long long *)take(sizeof(long long) * (P + 1));
    float *lam = (float *)take(sizeof(float) * P);
    const size_t described = used;
    D.Kt = (float *)take(sizeof(float) * (size_t)P * BMAX * BMAX);
    D.kpe = (double *)take(sizeof(double) * (size_t)tx);
    D.keq = (double *)take(sizeof(double) * (size_t)ty);
    D.landmarks = (float *)take(sizeof(float) * (size_t)P * (D.l > 0 ? D.l : 1) * d);
    D.buckets = (int *)take(sizeof(int) * (size_t)(D.R > 0 ? D.R : 1) * (tx + ty));
    D.log_u = (double *)take(sizeof(double) * (size_t)(tx + ty));
    D.log_v = (double *)take(sizeof(double) * (size_t)(tx + ty));
    D.counters = (unsigned long long *)take(64);
    h.ws_used = used;
    const size_t least = used;
    // Last, room for the marginals of a run.  It belongs to what a batch needs; a workspace that ends before it is still
    // taken, and the marginals are then formed when they are asked for.
    float *row_marg = (float *)take(sizeof(float) * (size_t)(tx + ty));
    float *col_marg = (float *)take(sizeof(float) * (size_t)(tx + ty));
    if (used <= workspace_bytes) {
        D.row_marg = row_marg;
        D.col_marg = col_marg;
        h.ws_used = used;
    }
    if (bytes_needed) *bytes_needed = used + 256;
    if (least > workspace_bytes) return LCN_ERR_ALLOC;
    D.x_off = xo;
    D.y_off = yo;
    D.lambda = lam;

    // the host block: the description as it lies in the workspace, then distances, residuals and marks
    const size_t result_bytes = (sizeof(double) * (size_t)P + 255) & ~(size_t)255;
    if (take_host_block(described + 2 * result_bytes + 256, h.host) != hipSuccess) {
        (void)hipGetLastError();
        return LCN_ERR_DEVICE;
    }
    char *host = h.host.ptr;
    memcpy(host + ((char *)xo - base), desc->x_off, sizeof(long long) * (P + 1));
    memcpy(host + ((char *)yo - base), desc->y_off, sizeof(long long) * (P + 1));
    memcpy(host + ((char *)lam - base), desc->lambda, sizeof(float) * P);
    D.dist = (double *)(host + described);
    D.resid = (double *)(host + described + result_bytes);
    D.marks = (int *)(host + described + 2 * result_bytes);
    D.marks[0] = D.marks[1] = 0;
    const long long words = (long long)(((char *)(lam + P) - base) / 4);
    hipLaunchKernelGGL(batch_upload_kernel, dim3((unsigned)((words + 255) / 256)), dim3(256), 0, h.stream,
                       (const unsigned *)host, (unsigned *)base, words, (unsigned *)D.counters, 16);
    BHIPCHK(hipGetLastError());
    BHIPCHK(launch_batched_build(h));
    BHIPCHK(hipStreamSynchronize(h.stream));
    if (*(volatile int *)D.marks) return LCN_ERR_SINGULAR;
    h.magic = BATCH_MAGIC;
    guard.p = nullptr;
    *out = (lcn_handle)hp;
    return LCN_OK;
}

lcn_status lcn_batched_results(lcn_handle hh, double *dist_host, double *resid_host, float *row_dev, float *col_dev)
{
    if (!is_batched_handle(hh)) return LCN_ERR_STATE;
    return batched_query(hh, dist_host, resid_host, row_dev, col_dev);
}

lcn_status lcn_batched_get(lcn_handle hh, double *log_u_dev, double *log_v_dev, float *landmarks_dev,
                           int32_t *buckets_dev, float *kernel_dev)
{
    if (!is_batched_handle(hh)) return LCN_ERR_STATE;
    BatchHandle &h = *(BatchHandle *)hh;
    const BatchDev &D = h.dev;
    const size_t tz = (size_t)(h.total_x + h.total_y);
    if (log_u_dev) BHIPCHK(hipMemcpyAsync(log_u_dev, D.log_u, sizeof(double) * tz, hipMemcpyDeviceToDevice, h.stream));
    if (log_v_dev) BHIPCHK(hipMemcpyAsync(log_v_dev, D.log_v, sizeof(double) * tz, hipMemcpyDeviceToDevice, h.stream));
    if (landmarks_dev && D.l > 0)
        BHIPCHK(hipMemcpyAsync(landmarks_dev, D.landmarks, sizeof(float) * (size_t)D.P * D.l * D.d,
                               hipMemcpyDeviceToDevice, h.stream));
    if (buckets_dev && D.R > 0)
        BHIPCHK(hipMemcpyAsync(buckets_dev, D.buckets, sizeof(int) * (size_t)D.R * tz, hipMemcpyDeviceToDevice,
                               h.stream));
    if (kernel_dev)
        BHIPCHK(hipMemcpyAsync(kernel_dev, D.Kt, sizeof(float) * (size_t)D.P * BMAX * BMAX, hipMemcpyDeviceToDevice,
                               h.stream));
    BHIPCHK(hipStreamSynchronize(h.stream));
    return LCN_OK;
}

lcn_status lcn_deletion_costs(const float *X, int64_t total, int32_t d, const float *alpha, float *out,
                              void *hip_stream)
{
    if (total < 0 || d < 1) return LCN_ERR_INVALID_ARG;
    if (total == 0) return LCN_OK;
    if (!X || !alpha || !out) return LCN_ERR_INVALID_ARG;
    const long long groups = (total + 255) / 256;
    if (groups > 0x7FFFFFFFLL) return LCN_ERR_INVALID_ARG;
    hipLaunchKernelGGL(deletion_cost_kernel, dim3((unsigned)groups), dim3(256), 0, (hipStream_t)hip_stream, X,
                       (long long)total, d, alpha, out);
    BHIPCHK(hipGetLastError());
    return LCN_OK;
}

lcn_status lcn_head_lambdas(float lambda, int32_t num_heads, float *out_host)
{
    if (!out_host || !(lambda > 0.f) || num_heads < 1 || num_heads > 64) return LCN_ERR_INVALID_ARG;
    for (int k = 1; k <= num_heads; ++k) {
        const float v = (float)(std::exp2((double)k - 0.5 * (double)num_heads) * (double)lambda);
        if (!(v > 0.f) || !std::isfinite(v)) return LCN_ERR_INVALID_ARG;
        out_host[k - 1] = v;
    }
    return LCN_OK;
}

}  // extern "C"
