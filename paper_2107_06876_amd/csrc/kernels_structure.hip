// Structure build: input conversion, exact-rule bucket assignment (k-means
// and cross-polytope hashing), the k-means centroid update, the bucket sort
// into blocks, and the CSR export.
//
// This file is compiled with -ffp-contract=off: the bucket of a point is
// decided by fp64 arithmetic evaluated in a fixed order with separate
// multiplies and adds, so that it is a function of the inputs alone.
#include "lcn_internal.h"

#pragma clang fp contract(off)

namespace lcn {

// ------------------------------------------------------------- conversion --

__global__ void convert_kernel(const void *X, long long nx_elems, const void *Y, long long total, int dtype, float *Z,
                               unsigned *range_flag)
{
    long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    long long stride = (long long)gridDim.x * blockDim.x;
    bool bad = false;
    for (; i < total; i += stride) {
        const void *src = i < nx_elems ? X : Y;
        long long j = i < nx_elems ? i : i - nx_elems;
        float v;
        if (dtype == LCN_BF16) {
            unsigned bits = ((const unsigned short *)src)[j];
            v = __uint_as_float(bits << 16);
        } else {
            v = ((const float *)src)[j];
        }
        Z[i] = v;
        bad |= !(fabsf(v) < 1024.0f);
    }
    if (bad) atomicOr(range_flag, 1u);
}

hipError_t launch_convert(const void *X, long long n, const void *Y, long long m, int d, int dtype, float *Z,
                          unsigned *range_flag, hipStream_t s)
{
    long long total = (n + m) * d;
    int grid = (int)((total + 255) / 256 < 4096 ? (total + 255) / 256 : 4096);
    hipLaunchKernelGGL(convert_kernel, dim3(grid), dim3(256), 0, s, X, n * d, Y, total, dtype, Z, range_flag);
    return hipGetLastError();
}

// Several small regions cleared by one launch (a clear of its own per region is a launch of its own,
// and a launch costs more than these clears).  Sizes in 4-byte words.
__global__ void clear_regions_kernel(ClearRegions R)
{
    for (int q = 0; q < R.count; ++q)
        for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < R.words[q];
             i += (long long)gridDim.x * blockDim.x)
            R.ptr[q][i] = 0u;
}

hipError_t launch_clear_regions(const ClearRegions &R, hipStream_t s)
{
    long long most = 0;
    for (int q = 0; q < R.count; ++q) most = R.words[q] > most ? R.words[q] : most;
    if (most <= 0) return hipSuccess;
    const long long blocks = (most + 255) / 256;
    hipLaunchKernelGGL(clear_regions_kernel, dim3((unsigned)(blocks < 1024 ? blocks : 1024)), dim3(256), 0, s, R);
    return hipGetLastError();
}

__global__ void gather_rows_kernel(const float *Z, int d, const long long *idx, int k, float *out)
{
    int c = blockIdx.x;
    const long long src = idx[c];   // negative: no such row, the slot is filled with zeros
    for (int j = threadIdx.x; j < d; j += blockDim.x) out[(long long)c * d + j] = src < 0 ? 0.f : Z[src * d + j];
}

hipError_t launch_gather_rows(const float *Z, int d, const long long *idx, int k, float *out, hipStream_t s)
{
    hipLaunchKernelGGL(gather_rows_kernel, dim3(k), dim3(128), 0, s, Z, d, idx, k, out);
    return hipGetLastError();
}

// ---------------------------------------------------- k-means++ seeding --
//
// Landmarks "sampled via k-means++" (Sec. 4): the first point uniformly, each
// further one with probability proportional to its squared distance w_i to
// the nearest point chosen so far.  The draw is integer work so that it has
// one answer: w_i by the fp64 bucket rule, weight q_i = floor(w_i 2^(38-e))
// where 4 max|z|^2 = f 2^e (1/2 <= f < 1) bounds every distance, pick = lowest
// i with q_0 + .. + q_i > r_t mod (sum q), r_t the t-th splitmix64 output.  A
// chosen point carries w = -1 (weight 0).  If the weights sum to 0 the lowest
// index not chosen yet is taken.
//
// One step = one sweep over the points (distance to the newest landmark,
// minimum, weights, per-workgroup totals) and one single-workgroup pick.

constexpr int PP_POINTS = 64;   // points per workgroup of the sweep: one wavefront, one point per lane
constexpr int PP_MAX_GROUPS = 16384;

__device__ inline int kmeanspp_shift(unsigned long long m2_bits)
{
    // 4 * m2 = f * 2^e with 1/2 <= f < 1: e = biased exponent - 1020 (m2 is 0 or a normal double)
    return 38 - ((int)((m2_bits >> 52) & 0x7FF) - 1020);
}

__device__ inline unsigned long long kmeanspp_weight(double w, int shift)
{
    return w > 0.0 ? (unsigned long long)floor(ldexp(w, shift)) : 0ull;
}

// MODE 0: largest squared norm of a point -> state[0] (bits of a non-negative double order like integers)
// MODE 1: w = D(z, c);  MODE 2: w = min(w, D(z, c));  both: partial[workgroup] = sum of the weights
// The wavefront reads its 64 rows in tiles of 32 dimensions (two rows per load instruction, all 32
// loads of a tile in flight together, the next tile's while this one is summed), turns the tile
// through LDS, and every lane adds up its own point's terms in dimension order.
template <int MODE>
__global__ __launch_bounds__(64) void kmeanspp_sweep_kernel(const float *Z, long long N, int d, const float *c,
                                                            const int *picks, int t, double *w,
                                                            unsigned long long *state, unsigned long long *partial)
{
    __shared__ float tile[64][33];
    __shared__ float csh[32];
    const int lane = threadIdx.x;
    const int half = lane >> 5, col = lane & 31;
    const long long i0 = (long long)blockIdx.x * PP_POINTS;
    // rows past the end repeat the last row (their lanes are dropped at the end)
    long long rowoff[32];
#pragma unroll
    for (int q = 0; q < 32; ++q) {
        const long long row = i0 + 2 * q + half;
        rowoff[q] = (row < N ? row : N - 1) * d;
    }
    float v[32];
    float cv = 0.f;
    auto fetch = [&](int k0) {
        const int kc = k0 + col < d ? k0 + col : d - 1;   // columns past the end repeat the last one (not summed)
#pragma unroll
        for (int q = 0; q < 32; ++q) v[q] = Z[rowoff[q] + kc];
        if (MODE != 0) cv = c[k0 + (lane & 31) < d ? k0 + (lane & 31) : d - 1];
    };
    fetch(0);
    double s = 0.0;
    for (int k0 = 0; k0 < d; k0 += 32) {
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 32; ++q) tile[2 * q + half][col] = v[q];
        if (lane < 32) csh[lane] = cv;
        __syncthreads();
        if (k0 + 32 < d) fetch(k0 + 32);
        const int kend = d - k0 < 32 ? d - k0 : 32;
        if (kend == 32) {
#pragma unroll
            for (int kk = 0; kk < 32; ++kk) {
                const double df = (double)tile[lane][kk] - (double)csh[kk];
                const double sq = df * df;
                s = s + sq;
            }
        } else {
            for (int kk = 0; kk < kend; ++kk) {
                const double df = (double)tile[lane][kk] - (double)csh[kk];
                const double sq = df * df;
                s = s + sq;
            }
        }
    }
    const long long i = i0 + lane;
    unsigned long long r = 0;
    if (MODE == 0) {
        r = i < N ? (unsigned long long)__double_as_longlong(s) : 0ull;
        for (int o = 32; o > 0; o >>= 1) {
            const unsigned long long other = __shfl_xor(r, o, 64);
            r = other > r ? other : r;
        }
        if (lane == 0) atomicMax(&state[0], r);
    } else {
        if (i < N) {
            double wn = s;
            if (MODE == 2) wn = fmin(w[i], s);
            if (i == (long long)picks[t]) wn = -1.0;
            w[i] = wn;
            r = kmeanspp_weight(wn, kmeanspp_shift(state[0]));
        }
        for (int o = 32; o > 0; o >>= 1) r += __shfl_xor(r, o, 64);
        if (lane == 0) partial[blockIdx.x] = r;
    }
}

// One workgroup of 1024 threads: the t-th pick from the per-workgroup totals of the sweep, its
// index into picks[t], its row into cent[t].  nb <= 16384 totals, sixteen per thread.
__global__ __launch_bounds__(1024) void kmeanspp_pick_kernel(const float *Z, long long N, int d, const double *w,
                                                             const unsigned long long *state,
                                                             const unsigned long long *partial, int nb,
                                                             const unsigned long long *rnd, int t, int *picks,
                                                             float *cent)
{
    __shared__ unsigned long long scan[1024];
    __shared__ long long found;     // index of the pick
    __shared__ long long blk;       // workgroup of the sweep that holds it
    __shared__ unsigned long long rem_sh;
    const int tid = threadIdx.x;
    if (tid == 0) {
        found = -1;
        blk = -1;
    }
    if (t == 0) {
        __syncthreads();
        if (tid == 0) found = (long long)(rnd[0] % (unsigned long long)N);
        __syncthreads();
    } else {
        unsigned long long v[16], local = 0;
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            const int b = tid * 16 + q;
            v[q] = b < nb ? partial[b] : 0ull;
            local += v[q];
        }
        scan[tid] = local;
        __syncthreads();
        for (int o = 1; o < 1024; o <<= 1) {   // inclusive scan
            const unsigned long long add = tid >= o ? scan[tid - o] : 0ull;
            __syncthreads();
            scan[tid] += add;
            __syncthreads();
        }
        const unsigned long long total = scan[1023];
        if (total == 0) {
            // every point left coincides with a chosen one: lowest index not chosen yet
            long long best = N;
            for (long long i = tid; i < N; i += 1024)
                if (w[i] >= 0.0 && i < best) best = i;
            __syncthreads();
            scan[tid] = (unsigned long long)best;
            __syncthreads();
            for (int o = 512; o > 0; o >>= 1) {
                if (tid < o && scan[tid + o] < scan[tid]) scan[tid] = scan[tid + o];
                __syncthreads();
            }
            if (tid == 0) found = (long long)scan[0];
            __syncthreads();
        } else {
            const unsigned long long target = rnd[t] % total;
            unsigned long long run = scan[tid] - local;   // total of the workgroups before this thread's sixteen
            if (local > 0 && run <= target && target < scan[tid]) {
                bool done = false;
#pragma unroll
                for (int q = 0; q < 16; ++q) {
                    if (!done && target < run + v[q]) {
                        blk = tid * 16 + q;
                        rem_sh = target - run;
                        done = true;
                    }
                    run += v[q];
                }
            }
            __syncthreads();
            const long long base = blk * PP_POINTS;
            const unsigned long long rem = rem_sh;
            const int shift = kmeanspp_shift(state[0]);
            unsigned long long q = 0;
            if (tid < PP_POINTS && base + tid < N) q = kmeanspp_weight(w[base + tid], shift);
            __syncthreads();
            scan[tid] = q;
            __syncthreads();
            for (int o = 1; o < PP_POINTS; o <<= 1) {
                const unsigned long long add = (tid >= o && tid < PP_POINTS) ? scan[tid - o] : 0ull;
                __syncthreads();
                if (tid < PP_POINTS) scan[tid] += add;
                __syncthreads();
            }
            if (tid < PP_POINTS && q > 0 && scan[tid] - q <= rem && rem < scan[tid]) found = base + tid;
            __syncthreads();
        }
    }
    const long long pick = found;
    if (pick < 0 || pick >= N) return;   // cannot happen; leaves picks[t] untouched rather than reading out of range
    if (tid == 0) picks[t] = (int)pick;
    for (int j = tid; j < d; j += 1024) cent[(long long)t * d + j] = Z[pick * d + j];
}

// k points of Z by k-means++ seeding into cent (k x d); rnd: k splitmix64 outputs (device);
// w: N doubles, partial: ceil(N / 64) totals, picks: k ints, state: one 64-bit word.
hipError_t launch_kmeanspp(const float *Z, long long N, int d, int k, const unsigned long long *rnd, double *w,
                           unsigned long long *partial, int *picks, unsigned long long *state, float *cent,
                           hipStream_t s)
{
    const int nb = (int)((N + PP_POINTS - 1) / PP_POINTS);
    if (nb > PP_MAX_GROUPS || k > N) return hipErrorInvalidValue;
    hipError_t e = hipMemsetAsync(state, 0, sizeof(unsigned long long), s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kmeanspp_sweep_kernel<0>, dim3(nb), dim3(64), 0, s, Z, N, d, (const float *)nullptr,
                       (const int *)nullptr, 0, (double *)nullptr, state, (unsigned long long *)nullptr);
    for (int t = 0; t < k; ++t) {
        hipLaunchKernelGGL(kmeanspp_pick_kernel, dim3(1), dim3(1024), 0, s, Z, N, d, (const double *)w,
                           (const unsigned long long *)state, (const unsigned long long *)partial, nb, rnd, t, picks,
                           cent);
        if (t + 1 == k) break;
        if (t == 0)
            hipLaunchKernelGGL(kmeanspp_sweep_kernel<1>, dim3(nb), dim3(64), 0, s, Z, N, d,
                               (const float *)(cent + (long long)t * d), (const int *)picks, t, w, state, partial);
        else
            hipLaunchKernelGGL(kmeanspp_sweep_kernel<2>, dim3(nb), dim3(64), 0, s, Z, N, d,
                               (const float *)(cent + (long long)t * d), (const int *)picks, t, w, state, partial);
    }
    return hipGetLastError();
}

// ------------------------------------------------- exact-rule assignment --
//
// A block takes 64 points and walks over all candidates (centroids, or
// projection columns) in tiles of 64; each thread keeps a 4 x 4 patch of fp64
// accumulators.  Every accumulator adds its terms in ascending dimension
// order, multiply and add separately, which is the rule the bucket of a point
// is defined by.  KIND 0: squared distance, arg-min (k-means).  KIND 1: dot
// product with the columns of a d x h matrix, arg-max over [g, -g]
// (cross-polytope hashing).

constexpr int TILE = 64;
constexpr int KCH = 32;
constexpr int LDT = TILE + 4;

template <int KIND>
__global__ __launch_bounds__(256) void assign_kernel(const float *__restrict__ Z, long long N, int d,
                                                     const float *__restrict__ C, int k, int32_t *__restrict__ out)
{
    __shared__ float Ps[KCH][LDT];
    __shared__ float Cs[KCH][LDT];
    __shared__ double red_v[TILE][17];
    __shared__ int red_i[TILE][17];
    __shared__ long long pidx[TILE];  // the 64 points of this workgroup (-1: none)

    const int tid = threadIdx.x;
    const int tx = tid & 15, ty = tid >> 4;
    const long long p0 = (long long)blockIdx.x * TILE;
    if (tid < TILE) pidx[tid] = p0 + tid < N ? p0 + tid : -1;
    __syncthreads();

    double bestv[4];
    int besti[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        bestv[i] = 0.0;
        besti[i] = -1;
    }

    for (int c0 = 0; c0 < k; c0 += TILE) {
        double acc[4][4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[i][j] = 0.0;

        for (int k0 = 0; k0 < d; k0 += KCH) {
            __syncthreads();
            // stage 64 points x 32 dims and 64 candidates x 32 dims, zero padded
            {
                const int kk = tid & 31;
                const int r0 = tid >> 5;
#pragma unroll
                for (int pass = 0; pass < 8; ++pass) {
                    int r = r0 + pass * 8;
                    long long p = pidx[r];
                    float v = 0.f;
                    if (p >= 0 && k0 + kk < d) v = Z[p * d + k0 + kk];
                    Ps[kk][r] = v;
                }
                if (KIND == 0) {
#pragma unroll
                    for (int pass = 0; pass < 8; ++pass) {
                        int r = r0 + pass * 8;
                        int c = c0 + r;
                        float v = 0.f;
                        if (c < k && k0 + kk < d) v = C[(long long)c * d + k0 + kk];
                        Cs[kk][r] = v;
                    }
                } else {
                    const int cc = tid & 63;
                    const int kr = tid >> 6;
#pragma unroll
                    for (int pass = 0; pass < 8; ++pass) {
                        int kq = kr + pass * 4;
                        float v = 0.f;
                        if (c0 + cc < k && k0 + kq < d) v = C[(long long)(k0 + kq) * k + c0 + cc];
                        Cs[kq][cc] = v;
                    }
                }
            }
            __syncthreads();
#pragma unroll 4
            for (int kk = 0; kk < KCH; ++kk) {
                const float4 pz = *(const float4 *)&Ps[kk][ty * 4];
                const float4 cz = *(const float4 *)&Cs[kk][tx * 4];
                const double pv[4] = {(double)pz.x, (double)pz.y, (double)pz.z, (double)pz.w};
                const double cv[4] = {(double)cz.x, (double)cz.y, (double)cz.z, (double)cz.w};
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        if (KIND == 0) {
                            double t = pv[i] - cv[j];
                            double t2 = t * t;
                            acc[i][j] = acc[i][j] + t2;
                        } else {
                            double t = pv[i] * cv[j];
                            acc[i][j] = acc[i][j] + t;
                        }
                    }
            }
        }
        // fold this tile's candidates into the running best (lowest index wins ties)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            int c = c0 + tx * 4 + j;
            if (c >= k) continue;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (KIND == 0) {
                    double D = acc[i][j];
                    if (besti[i] < 0 || D < bestv[i] || (D == bestv[i] && c < besti[i])) {
                        bestv[i] = D;
                        besti[i] = c;
                    }
                } else {
                    double g = acc[i][j];
                    // candidate c has value g, candidate k + c has value -g
                    if (besti[i] < 0 || g > bestv[i] || (g == bestv[i] && c < besti[i])) {
                        bestv[i] = g;
                        besti[i] = c;
                    }
                    double ng = -g;
                    if (ng > bestv[i] || (ng == bestv[i] && k + c < besti[i])) {
                        bestv[i] = ng;
                        besti[i] = k + c;
                    }
                }
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        red_v[ty * 4 + i][tx] = bestv[i];
        red_i[ty * 4 + i][tx] = besti[i];
    }
    __syncthreads();
    if (tid < TILE) {
        double bv = 0.0;
        int bi = -1;
        for (int t = 0; t < 16; ++t) {
            double v = red_v[tid][t];
            int ix = red_i[tid][t];
            if (ix < 0) continue;
            bool better;
            if (KIND == 0)
                better = bi < 0 || v < bv || (v == bv && ix < bi);
            else
                better = bi < 0 || v > bv || (v == bv && ix < bi);
            if (better) {
                bv = v;
                bi = ix;
            }
        }
        if (pidx[tid] >= 0) out[pidx[tid]] = bi;
    }
}

// Exact rule on what the filter left undecided, in one launch.
//
// Points with more than two candidates (the list): one workgroup per point, one thread per centroid (strided), each
// adding the dimensions left to right.  The centroids come through LDS, 32 dimensions of 256 of them (or 128 of 64) at a time in
// whole lines, the next ones already requested (a thread that reads its centroid's row by itself asks for 64 lines per
// load: 17 us for a few hundred points of 300 dimensions).
//
// Points with two candidates: sixteen per workgroup at a time.  The order of the additions is the rule, but the squares
// are independent of each other: the workgroup forms them for 64 dimensions of 32 (point, centroid) pairs with whole
// lines of the two rows, and a lane per pair adds them up from LDS, the next 64 dimensions already requested.  (A thread
// that reads both rows by itself waits ten times for memory: 17 us at 38 768 points of 300 dimensions.)
constexpr int UP = 32, UD = 64;   // pairs of a point and a centroid, dimensions
constexpr int UV = 8192;          // values of the centroids at a time for a listed point

union UndecidedRoom {
    float cent[UV + 128];   // [UL][UC + 1]
    double sq[UP][UD + 1];
};

// One listed point: UL dimensions of UC = UV / UL centroids at a time.
template <int UL>
__device__ inline void undecided_point(const float *__restrict__ z, int d, const float *__restrict__ C, int k, UndecidedRoom &room,
                                       float (*zs)[128], double &bv, int &bi)
{
    constexpr int UC = UV / UL, STEP = 256 / UL;
    float(*cent)[UC + 1] = reinterpret_cast<float(*)[UC + 1]>(room.cent);
    const int dim = threadIdx.x & (UL - 1), r0 = threadIdx.x / UL;
    for (int c0 = 0; c0 < k; c0 += UC) {
        const int c = c0 + (int)threadIdx.x;
        const bool mine = (int)threadIdx.x < UC;
        double s = 0.0;
        float cv[32], zv;
        auto fetch = [&](int j0) {   // past the last dimension or centroid: the last one again, not added
            const int j = j0 + dim < d ? j0 + dim : d - 1;
#pragma unroll
            for (int u = 0; u < 32; ++u) {
                const int r = c0 + r0 + STEP * u < k ? c0 + r0 + STEP * u : k - 1;
                cv[u] = C[(long long)r * d + j];
            }
            zv = z[j];
        };
        fetch(0);
        for (int j0 = 0; j0 < d; j0 += UL) {
            const int buf = (j0 / UL) & 1;
            __syncthreads();   // the dimensions before have been added
#pragma unroll
            for (int u = 0; u < 32; ++u) cent[dim][r0 + STEP * u] = cv[u];
            if (threadIdx.x < UL) zs[buf][dim] = zv;
            __syncthreads();
            fetch(j0 + UL);
            const int m = d - j0 < UL ? d - j0 : UL;
            if (mine) {
                if (m == UL) {
#pragma unroll 32
                    for (int e = 0; e < UL; ++e) {
                        const double t = (double)zs[buf][e] - (double)cent[e][threadIdx.x];
                        const double t2 = t * t;
                        s = s + t2;
                    }
                } else {
                    for (int e = 0; e < m; ++e) {
                        const double t = (double)zs[buf][e] - (double)cent[e][threadIdx.x];
                        const double t2 = t * t;
                        s = s + t2;
                    }
                }
            }
        }
        if (mine && c < k && (bi < 0 || s < bv)) {  // ascending c: strict < keeps the lowest index
            bv = s;
            bi = c;
        }
    }
}

template <int UL>
__global__ __launch_bounds__(256) void assign_undecided_kernel(const float *__restrict__ Z, int d, KmRuns R)
{
    const KmRun &run = R.run[blockIdx.y];
    const float *__restrict__ C = run.cent;
    const int k = run.k;
    int32_t *__restrict__ out = run.assign;
    const int *__restrict__ list = run.flagged, *__restrict__ pairs = run.pairs, *__restrict__ count = run.nflagged;
    __shared__ double bv_sh[256];
    __shared__ int bi_sh[256];
    __shared__ float zs[2][128];
    __shared__ UndecidedRoom room;
    auto &sq = room.sq;
    const int cnt = count[0];
    const long long npairs = count[1];
    for (int it = blockIdx.x; it < cnt; it += gridDim.x) {
        const long long p = list[it];
        double bv = 0.0;
        int bi = -1;
        undecided_point<UL>(Z + p * d, d, C, k, room, zs, bv, bi);
        bv_sh[threadIdx.x] = bv;
        bi_sh[threadIdx.x] = bi;
        __syncthreads();
        for (int o = 128; o > 0; o >>= 1) {
            if (threadIdx.x < o) {
                const double v2 = bv_sh[threadIdx.x + o];
                const int i2 = bi_sh[threadIdx.x + o];
                const double v1 = bv_sh[threadIdx.x];
                const int i1 = bi_sh[threadIdx.x];
                if (i2 >= 0 && (i1 < 0 || v2 < v1 || (v2 == v1 && i2 < i1))) {
                    bv_sh[threadIdx.x] = v2;
                    bi_sh[threadIdx.x] = i2;
                }
            }
            __syncthreads();
        }
        if (threadIdx.x == 0) out[p] = bi_sh[0];
    }
    // the workgroups without a listed point first
    for (long long s0 = (long long)(gridDim.x - 1 - blockIdx.x) * UP; s0 < 2 * npairs; s0 += (long long)gridDim.x * UP) {
        const int lane = threadIdx.x & 63;
        const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        // wavefront w forms the squares of slots 8 w .. 8 w + 7, lane j dimension j (past the last slot: the last again)
        const float *zr[UP / 4], *cr[UP / 4];
#pragma unroll
        for (int u = 0; u < UP / 4; ++u) {
            long long t = s0 + (UP / 4) * wave + u;
            t = t < 2 * npairs ? t : 2 * npairs - 1;
            zr[u] = Z + (long long)pairs[3 * (t >> 1)] * d;
            cr[u] = C + (long long)pairs[3 * (t >> 1) + 1 + (int)(t & 1)] * d;
        }
        float zv[UP / 4], cv[UP / 4];
        auto fetch = [&](int j0) {
            const int j = j0 + lane < d ? j0 + lane : d - 1;
#pragma unroll
            for (int u = 0; u < UP / 4; ++u) {
                zv[u] = zr[u][j];
                cv[u] = cr[u][j];
            }
        };
        double s = 0.0;
        fetch(0);
        for (int j0 = 0; j0 < d; j0 += UD) {
            __syncthreads();   // the sums of the dimensions before have been taken
#pragma unroll
            for (int u = 0; u < UP / 4; ++u) {
                const double t = (double)zv[u] - (double)cv[u];
                sq[(UP / 4) * wave + u][lane] = t * t;
            }
            __syncthreads();
            fetch(j0 + UD);
            if (threadIdx.x < UP) {
                const int m = d - j0 < UD ? d - j0 : UD;
                if (m == UD) {
#pragma unroll 16
                    for (int e = 0; e < UD; ++e) s = s + sq[threadIdx.x][e];
                } else {
                    for (int e = 0; e < m; ++e) s = s + sq[threadIdx.x][e];
                }
            }
        }
        if (threadIdx.x < UP) {   // neighbouring lanes hold a point's two candidates: the lower index if equal
            long long t = s0 + threadIdx.x;
            const bool live = t < 2 * npairs;
            t = live ? t : 2 * npairs - 1;
            const int c = pairs[3 * (t >> 1) + 1 + (int)(t & 1)];
            const double so = __shfl_xor(s, 1, 64);
            const int co = __shfl_xor(c, 1, 64);
            if (live && (t & 1) == 0) out[pairs[3 * (t >> 1)]] = (so < s || (so == s && co < c)) ? co : c;
        }
    }
}

hipError_t launch_assign_undecided(const float *Z, int d, const KmRuns &runs, hipStream_t s)
{
    const dim3 grid(1024, (unsigned)runs.count);
    // What bounds a listed point is a trip to memory per UL dimensions: wide rows are taken 128 dimensions at a time if the
    // centroids are few enough (6000 points of 1000 dimensions, 40 centroids: 31 us instead of 38; up to 512 dimensions the
    // shorter trips are as good).  Such runs come one at a time.
    if (d > 512 && runs.run[0].k <= UV / 128)
        hipLaunchKernelGGL(assign_undecided_kernel<128>, grid, dim3(256), 0, s, Z, d, runs);
    else
        hipLaunchKernelGGL(assign_undecided_kernel<32>, grid, dim3(256), 0, s, Z, d, runs);
    return hipGetLastError();
}

hipError_t launch_assign_kmeans(const float *Z, long long N, int d, const float *cent, int k, int32_t *out, hipStream_t s)
{
    int grid = (int)((N + TILE - 1) / TILE);
    hipLaunchKernelGGL(assign_kernel<0>, dim3(grid), dim3(256), 0, s, Z, N, d, cent, k, out);
    return hipGetLastError();
}

hipError_t launch_assign_crosspolytope(const float *Z, long long N, int d, const float *Rm, int b, int32_t *out,
                                       hipStream_t s)
{
    int grid = (int)((N + TILE - 1) / TILE);
    hipLaunchKernelGGL(assign_kernel<1>, dim3(grid), dim3(256), 0, s, Z, N, d, Rm, b / 2, out);
    return hipGetLastError();
}

// ------------------------------------------- hierarchical k-means, AND hash --
//
// Lower levels of hierarchical k-means hashing (App. "Choosing LSH neighbors and
// Nystrom landmarks"): inside every cluster of the level above, a k-means of its
// own.  The points arrive grouped by parent (`order`), cut into chunks of at most
// 64 members of ONE parent: chunk = {parent, first position in order, members}.
// A wavefront takes a chunk, one member per lane, and adds up the squared
// distances to all children of that parent at once (children's centroids in
// LDS, read as broadcasts) -- the bucket rule: fp64, dimensions in order,
// multiply and add separately, lowest index among the minima.  bucket =
// parent * branch + child.
constexpr int HK_MAX_BRANCH = 32;

// Children's centroids as fp64, laid out [parent][dimension][child] with the children padded to
// `brp` (4, 8, 16 or 32): the sweep below reads one dimension of all children of a parent as one
// run of wave-uniform (scalar) loads.  A child that does not exist gets +infinity, which no
// minimum picks.
__global__ void children_layout_kernel(const float *cent, int d, int branch, int brp, const int *nchild,
                                       long long total, double *out)
{
    const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= total) return;
    const int j = (int)(e % brp);
    const long long pk = e / brp;
    const int k = (int)(pk % d);
    const long long parent = pk / d;
    out[e] = j < nchild[parent] ? (double)cent[(parent * branch + j) * d + k] : INFINITY;
}

template <int BRP>
__global__ __launch_bounds__(64) void assign_children_kernel(const float *Z, int d, const double *centT, int branch,
                                                             const int *order, const int *chunks, int32_t *out)
{
    __shared__ float tile[64][33];
    __shared__ int mem_sh[64];
    const int lane = threadIdx.x;
    const int half = lane >> 5, col = lane & 31;
    const int parent = __builtin_amdgcn_readfirstlane(chunks[3 * blockIdx.x]);
    const int first = chunks[3 * blockIdx.x + 1], cnt = chunks[3 * blockIdx.x + 2];
    const int me = order[first + (lane < cnt ? lane : cnt - 1)];   // lanes past the end repeat the last member
    mem_sh[lane] = me;
    __syncthreads();
    long long rowoff[32];
#pragma unroll
    for (int q = 0; q < 32; ++q) rowoff[q] = (long long)mem_sh[2 * q + half] * d;
    // wave-uniform address in the constant address space: read through the scalar unit
    typedef const __attribute__((address_space(4))) double *cptr;
    cptr ct = (cptr)(unsigned long long)(centT + (long long)parent * d * BRP);
    double acc[BRP];
#pragma unroll
    for (int j = 0; j < BRP; ++j) acc[j] = 0.0;
    float v[32];
    auto fetch = [&](int k0) {
        const int kc = k0 + col < d ? k0 + col : d - 1;
#pragma unroll
        for (int q = 0; q < 32; ++q) v[q] = Z[rowoff[q] + kc];
    };
    fetch(0);
    for (int k0 = 0; k0 < d; k0 += 32) {
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 32; ++q) tile[2 * q + half][col] = v[q];
        __syncthreads();
        if (k0 + 32 < d) fetch(k0 + 32);
        const int kend = d - k0 < 32 ? d - k0 : 32;
        for (int kk = 0; kk < kend; ++kk) {
            const double zv = (double)tile[lane][kk];
            cptr crow = ct + (long long)(k0 + kk) * BRP;
#pragma unroll
            for (int j = 0; j < BRP; ++j) {
                const double df = zv - crow[j];
                const double sq = df * df;
                acc[j] = acc[j] + sq;
            }
        }
    }
    int best = 0;
    double bestD = acc[0];
#pragma unroll
    for (int j = 1; j < BRP; ++j) {
        if (acc[j] < bestD) {
            bestD = acc[j];
            best = j;
        }
    }
    if (lane < cnt) out[me] = parent * branch + best;
}

// centT: scratch of parents * d * 32 doubles at most
hipError_t launch_assign_children(const float *Z, int d, const float *cent, long long parents, int branch,
                                  const int *nchild, const int *order, const int *chunks, int nchunks, double *centT,
                                  int32_t *out, hipStream_t s)
{
    if (branch < 1 || branch > HK_MAX_BRANCH) return hipErrorInvalidValue;
    if (nchunks < 1) return hipSuccess;
    const int brp = branch <= 4 ? 4 : branch <= 8 ? 8 : branch <= 16 ? 16 : 32;
    const long long total = parents * d * brp;
    hipLaunchKernelGGL(children_layout_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, cent, d, branch,
                       brp, nchild, total, centT);
#define LCN_CHILDREN(B)                                                                                          \
    hipLaunchKernelGGL(assign_children_kernel<B>, dim3(nchunks), dim3(64), 0, s, Z, d, (const double *)centT, branch, \
                       order, chunks, out)
    if (brp == 4) LCN_CHILDREN(4);
    else if (brp == 8) LCN_CHILDREN(8);
    else if (brp == 16) LCN_CHILDREN(16);
    else LCN_CHILDREN(32);
#undef LCN_CHILDREN
    return hipGetLastError();
}

// AND construction: the bucket of a band of hashes is the tuple of their values,
// numbered acc * b + h, one hash at a time.
__global__ void combine_hash_kernel(int32_t *acc, const int32_t *h, int b, int first, long long N)
{
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < N) acc[i] = (first ? 0 : acc[i] * b) + h[i];
}

hipError_t launch_combine_hash(int32_t *acc, const int32_t *h, int b, int first, long long N, hipStream_t s)
{
    hipLaunchKernelGGL(combine_hash_kernel, dim3((unsigned)((N + 255) / 256)), dim3(256), 0, s, acc, h, b, first, N);
    return hipGetLastError();
}

// -------------------------------------------------------- k-means update --
//
// Member sums in 2^-32 fixed point: integer addition is associative, so the
// sums are the same in any order.  Two ways to them:
//
// By members (few clusters times points): a workgroup takes ONE cluster and a range of at most 8192 points, reads
// that range's assignments, keeps the indices of its members in LDS and adds up their rows.  One range: the new
// centroid follows in the same launch; several: a second launch adds up the ranges' sums.  Every workgroup of a range
// reads the same assignments (from the cache, 4 k N bytes in all).
//
// Otherwise a counting sort of the points by cluster first:
//   count   -- members per cluster (histogram in LDS, one device atomic per
//              workgroup and cluster present);
//   scatter -- point indices grouped by cluster (each workgroup redoes the
//              small scan of the counts, reserves its ranges with one atomic per
//              cluster present and ranks its points in LDS);
//   partial, mean -- see there (rows of more than 512 dimensions: sum).
// The count and cursor arrays exist twice and alternate between updates: the last
// kernel clears the pair the next update will use.
//
// Whoever writes a centroid also writes its bf16 planes and squared norm for the next assignment step.

constexpr int KM_POINTS = 2048;  // points per workgroup of count and scatter

__device__ inline void write_centroid(const KmRun &P, int c, int d, int j, float v)
{
    P.cent[(long long)c * d + j] = v;
    if (P.first) {   // operand order: groups of 32 rows, steps of 16 dimensions, lane = row % 32 + 32 (j % 16 / 8)
        const long long at = (((long long)(c >> 5) * ((d + 15) / 16) + (j >> 4)) * 64 + (c & 31) + 32 * (j >> 3 & 1)) * 8 + (j & 7);
        const unsigned h = bf16_bits(v);
        P.first[at] = (unsigned short)h;
        P.first[P.plane + at] = (unsigned short)bf16_bits(v - __uint_as_float(h << 16));   // the difference is exact
    }
}

// The centroid's squared norm from every thread's share of it; sh: a double per wavefront of the workgroup.
__device__ inline void write_norm(const KmRun &P, int c, double sq, double *sh)
{
    for (int o = 1; o < 64; o <<= 1) sq += __shfl_xor(sq, o, 64);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = sq;
    __syncthreads();
    if (threadIdx.x == 0 && P.first) {
        double s = 0.0;
        for (int w = 0; w < (int)(blockDim.x >> 6); ++w) s += sh[w];
        P.cn[c] = (float)s;
    }
}

__global__ __launch_bounds__(256) void kmeans_count_kernel(const int32_t *__restrict__ assign, long long N, int k,
                                                           int *__restrict__ counts)
{
    extern __shared__ int hist[];  // k
    for (int t = threadIdx.x; t < k; t += 256) hist[t] = 0;
    __syncthreads();
    const long long p0 = (long long)blockIdx.x * KM_POINTS;
    for (int q = threadIdx.x; q < KM_POINTS; q += 256)
        if (p0 + q < N) atomicAdd(&hist[assign[p0 + q]], 1);
    __syncthreads();
    for (int t = threadIdx.x; t < k; t += 256)
        if (hist[t]) atomicAdd(&counts[t], hist[t]);
}

__global__ __launch_bounds__(256) void kmeans_scatter_kernel(const int32_t *__restrict__ assign, long long N, int k,
                                                             const int *__restrict__ counts, int *__restrict__ cursor,
                                                             int *__restrict__ order, int *__restrict__ offs)
{
    extern __shared__ int sh[];  // start[k] (where this workgroup's members of a cluster go), hist[k]
    __shared__ int part[256];
    int *start = sh, *hist = sh + k;
    const int tid = threadIdx.x;
    // exclusive scan of the counts: a contiguous run per thread, then the 256 run totals
    const int seg = (k + 255) / 256;
    const int lo = tid * seg, hi = lo + seg < k ? lo + seg : k;
    int run = 0;
    for (int t = lo; t < hi; ++t) run += counts[t];
    part[tid] = run;
    for (int t = tid; t < k; t += 256) hist[t] = 0;
    __syncthreads();
    if (tid == 0) {
        int acc = 0;
        for (int t = 0; t < 256; ++t) {
            const int v = part[t];
            part[t] = acc;
            acc += v;
        }
    }
    __syncthreads();
    run = part[tid];
    for (int t = lo; t < hi; ++t) {
        start[t] = run;
        if (blockIdx.x == 0) offs[t] = run;  // where each cluster's members begin, for the sum kernel
        run += counts[t];
    }
    __syncthreads();
    const long long p0 = (long long)blockIdx.x * KM_POINTS;
    int rank[KM_POINTS / 256], cl[KM_POINTS / 256];
#pragma unroll
    for (int u = 0; u < KM_POINTS / 256; ++u) {
        const long long p = p0 + tid + 256 * u;
        cl[u] = p < N ? assign[p] : -1;
        rank[u] = cl[u] >= 0 ? atomicAdd(&hist[cl[u]], 1) : 0;
    }
    __syncthreads();
    for (int t = tid; t < k; t += 256)
        if (hist[t]) start[t] += atomicAdd(&cursor[t], hist[t]);
    __syncthreads();
#pragma unroll
    for (int u = 0; u < KM_POINTS / 256; ++u)
        if (cl[u] >= 0) order[start[cl[u]] + rank[u]] = (int)(p0 + tid + 256 * u);
}

// grid: (k, ceil(d / SW)); 1024 threads.  SW = 64: a wave-wide load is one member's 64 dimensions.
// SW = 16 (few clusters: more, narrower workgroups): it is 16 dimensions of four members.
template <int SW, int WPB>
__global__ __launch_bounds__(64 * WPB) void kmeans_sum_kernel(const float *__restrict__ Z, int d, int k,
                                                          const int *__restrict__ counts, const int *__restrict__ offs,
                                                          const int *__restrict__ order, float *__restrict__ cent,
                                                          int *__restrict__ counts_next, int *__restrict__ cursor_next,
                                                          int *reset)
{
    constexpr int RPL = 64 / SW;   // members per wave-wide load
    __shared__ long long red[WPB][SW];
    const int c = blockIdx.x, slice = blockIdx.y;
    const int lane = threadIdx.x & 63;
    const int sub = lane / SW, jl = lane % SW;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (slice == 0 && threadIdx.x == 0) {  // scratch of the next assignment and update steps starts from zero
        counts_next[c] = 0;
        cursor_next[c] = 0;
        if (c == 0 && reset) {
            reset[0] = 0;
            reset[1] = 0;
        }
    }
    const int cnt = counts[c];
    const int *__restrict__ mem = order + offs[c];
    const int j = SW * slice + jl;
    const bool jin = j < d;
    long long sum = 0;
    // the 16 wavefronts share out the members in contiguous runs; a wave reads up to 64 member
    // indices at once (one per lane) and then requests 16 loads before the first is added
    const int per = (cnt + WPB - 1) / WPB;
    const int beg = wave * per;
    const int end = beg + per < cnt ? beg + per : cnt;
    for (int base = beg; base < end; base += 64) {
        const int nloc = end - base < 64 ? end - base : 64;
        const int myidx = lane < nloc ? mem[base + lane] : 0;
        for (int u0 = 0; u0 < nloc; u0 += 16 * RPL) {
            float z[16];
#pragma unroll
            for (int u = 0; u < 16; ++u) {
                const int uu = u0 + u * RPL + sub;
                long long row;
                if (RPL == 1)
                    row = __builtin_amdgcn_readlane(myidx, uu < 64 ? uu : 63);
                else
                    row = __shfl(myidx, uu < 64 ? uu : 63, 64);
                // an unconditional load (a slot beyond the run reads row 0, a lane beyond the row's end
                // its last entry) keeps all sixteen in flight; what does not count is zeroed afterwards
                const float v = Z[row * d + (jin ? j : d - 1)];
                z[u] = (uu < nloc && jin) ? v : 0.f;
            }
#pragma unroll
            for (int u = 0; u < 16; ++u) sum += __double2ll_rn((double)z[u] * 4294967296.0);
        }
    }
    for (int o = SW; o < 64; o <<= 1) sum += __shfl_xor(sum, o, 64);   // the members a load held side by side
    if (lane < SW) red[wave][lane] = sum;
    __syncthreads();
    if (wave == 0 && lane < SW && jin && cnt > 0) {  // an empty cluster keeps its centroid
        long long tot = 0;
#pragma unroll
        for (int w = 0; w < WPB; ++w) tot += red[w][lane];
        const double mean = ((double)tot * (1.0 / 4294967296.0)) / (double)cnt;
        cent[(long long)c * d + j] = (float)mean;
    }
}

// Rows of up to 512 dimensions: the sums are taken in two steps that do not depend on how the members
// are spread over the clusters.  The member list (grouped by cluster) is cut into chunks of M
// consecutive entries, one wavefront per chunk; the wavefront reads whole rows (lane j holds dimensions
// j, 64 + j, ...: every line of a row is fetched once, eight rows requested before the first is added)
// and, whenever the cluster changes and at its end, writes the sums so far as a partial: chunk g's
// part of cluster c goes to slot g + c, which no other pair shares (chunks and clusters both advance
// along the list).  One workgroup per cluster then adds the partials of the chunks its members lie in
// and writes the mean.  No atomics, every launch as long as the others whatever the cluster sizes.
// The fixed-point value of an entry: z 2^32 + 1.5 2^52 rounds to an integer (to nearest even, as rint
// does) whose low mantissa bits are that integer in two's complement, so the bit patterns are added
// as they are and the constants' share is taken off per member (all modulo 2^64).
constexpr int KM_RANGE = 8192;   // points a workgroup looks through for its cluster's members
// Clusters times points up to which every cluster's workgroups look through the assignments themselves.  The clusters are
// those of all runs of a build: its runs look through their assignments at the same time, from the same caches.
// Build times, by members / counting and scattering (us), by millions of clusters times points: 24 (40 000 points, a run of 510
// clusters and one of 200) 1870 / 1940, 46 (40 000, two of 512 and 128) 2120 / 2200, 44 (60 000, two of 270 and 200) 2050 / 2110,
// 49 (60 000, 760 and 64) 1490 / 1530; 101 (60 000, two of 780 and 128) 3140 / 2930, 107 (100 000, three of 270 and 256)
// 5000 / 4800, 128 (80 000, four of 400) 3930 / 3520.  Up to 2^14 points, two ranges, whatever the clusters (at most 4096 of
// a run): 8000 points, five of 2000 2180 / 3070, 16 000, three of 2000 2530 / 2560.  And twice as much for more rounds than
// lanes, which only then can advance together: 72 (60 000, six of 200) 4050 / 4260, 74 (40 000, eight of 200 and 256) 4670 / 5100.
constexpr long long KM_MEMBERS_WORK = 1ll << 26, KM_MEMBERS_POINTS = 1ll << 14;

static int kmeans_ranges(long long N) { return (int)((N + KM_RANGE - 1) / KM_RANGE); }

bool kmeans_by_members(long long N, long long clusters, int d, bool more_than_lanes)
{
    return d <= 512 && (N <= KM_MEMBERS_POINTS || clusters * N <= (more_than_lanes ? 2 : 1) * KM_MEMBERS_WORK);
}

int kmeans_sum_chunk(long long N) { return N <= 65536 ? 16 : N <= 131072 ? 32 : N <= 262144 ? 64 : 128; }

size_t kmeans_partial_elems(long long N, int kmax, int d, bool members, bool sorted)
{
    if (d > 512) return 1;   // wider rows take the sliced kernel, which needs none
    // (4096 clusters of 2^14 points are 2^26 as well; kmax may be the buckets of a hash that is not k-means)
    const long long k = KM_MEMBERS_WORK / N < kmax ? KM_MEMBERS_WORK / N : kmax;
    const int M = kmeans_sum_chunk(N);
    const size_t by_members = members ? (size_t)k * (size_t)kmeans_ranges(N) : 0, by_sort = sorted ? (size_t)((N + M - 1) / M + kmax) : 0;
    return (by_members > by_sort ? by_members : by_sort) * (size_t)d;
}

constexpr unsigned long long FIX_MAGIC_BITS = 0x4338000000000000ull;   // 1.5 * 2^52

template <int NS>
__global__ __launch_bounds__(256) void kmeans_partial_kernel(const float *__restrict__ Z, long long N, int d, int M,
                                                             const int32_t *__restrict__ assign,
                                                             const int *__restrict__ order,
                                                             unsigned long long *__restrict__ part)
{
    const int lane = threadIdx.x & 63;
    const long long g = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
    const long long first = g * M;
    if (first >= N) return;
    const int mine = N - first < M ? (int)(N - first) : M;
    unsigned long long sum[NS];
#pragma unroll
    for (int q = 0; q < NS; ++q) sum[q] = 0ull;
    int cur = -1, held = 0;
    auto flush = [&]() {
        unsigned long long *dst = part + (size_t)(g + cur) * (size_t)d;
#pragma unroll
        for (int q = 0; q < NS; ++q) {
            const int j = 64 * q + lane;
            if (j < d) dst[j] = sum[q] - (unsigned long long)held * FIX_MAGIC_BITS;
            sum[q] = 0ull;
        }
        held = 0;
    };
    // Every load below is unconditional: a lane beyond the row's end re-reads the row's last entry and
    // a slot beyond the chunk's end the chunk's last member (what they add is never stored), so the
    // forty loads of eight rows are in flight together.
    int jc[NS];
#pragma unroll
    for (int q = 0; q < NS; ++q) jc[q] = 64 * q + lane < d ? 64 * q + lane : d - 1;
    auto add_row = [&](const float (&zr)[NS]) {
        ++held;
#pragma unroll
        for (int q = 0; q < NS; ++q)
            sum[q] += (unsigned long long)__double_as_longlong(fma((double)zr[q], 4294967296.0, 6755399441055744.0));
    };
    for (int base = 0; base < mine; base += 64) {
        const int nloc = mine - base < 64 ? mine - base : 64;
        const int at = lane < nloc ? lane : nloc - 1;
        const int myidx = order[first + base + at];
        const int mycl = assign[myidx];
        for (int u0 = 0; u0 < nloc; u0 += 8) {
            float z[8][NS];
            int cl[8];
            bool same = u0 + 8 <= nloc;
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int uu = u0 + u < nloc ? u0 + u : nloc - 1;
                const float *__restrict__ zrow = Z + (long long)__builtin_amdgcn_readlane(myidx, uu) * d;
                cl[u] = __builtin_amdgcn_readlane(mycl, uu);
                same = same && cl[u] == cur;
#pragma unroll
                for (int q = 0; q < NS; ++q) z[u][q] = zrow[jc[q]];
            }
            if (same) {   // the usual case: eight more members of the current cluster
#pragma unroll
                for (int u = 0; u < 8; ++u) add_row(z[u]);
            } else {
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    if (u0 + u < nloc) {   // the same in every lane
                        if (cl[u] != cur) {
                            if (cur >= 0) flush();
                            cur = cl[u];
                        }
                        add_row(z[u]);
                    }
                }
            }
        }
    }
    if (cur >= 0) flush();
}

// One workgroup of eight wavefronts per cluster: the wavefronts share out the chunks the cluster's
// members lie in, four chunks' partials (whole rows, lane j dimensions j, 64 + j, ...) requested
// together; a chunk index beyond the last is clamped and its row not added.
template <int NS>
__global__ __launch_bounds__(512) void kmeans_mean_kernel(const unsigned long long *__restrict__ part, int d, int M,
                                                          const int *__restrict__ counts,
                                                          int *__restrict__ counts_next,
                                                          int *__restrict__ cursor_next, KmRun run)
{
    const int *__restrict__ offs = run.offs;
    int *reset = run.keep_counts ? nullptr : run.nflagged;
    __shared__ unsigned long long red[8][NS][64];
    __shared__ double norm_sh[8];
    const int c = blockIdx.x;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (threadIdx.x == 0) {  // scratch of the next assignment and update steps starts from zero
        counts_next[c] = 0;
        cursor_next[c] = 0;
        if (c == 0 && reset) {
            reset[0] = 0;
            reset[1] = 0;
        }
    }
    const int cnt = counts[c];
    if (cnt == 0) return;  // an empty cluster keeps its centroid (the same in every thread)
    const int g0 = offs[c] / M, g1 = (offs[c] + cnt - 1) / M;
    int jc[NS];
    unsigned long long sum[NS];
#pragma unroll
    for (int q = 0; q < NS; ++q) {
        jc[q] = 64 * q + lane < d ? 64 * q + lane : d - 1;
        sum[q] = 0ull;
    }
    for (int g = g0 + wave; g <= g1; g += 32) {
        unsigned long long v[4][NS];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int gg = g + 8 * u <= g1 ? g + 8 * u : g1;
            const unsigned long long *__restrict__ row = part + (size_t)(gg + c) * (size_t)d;
#pragma unroll
            for (int q = 0; q < NS; ++q) v[u][q] = row[jc[q]];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (g + 8 * u <= g1) {   // the same in every lane
#pragma unroll
                for (int q = 0; q < NS; ++q) sum[q] += v[u][q];
            }
    }
#pragma unroll
    for (int q = 0; q < NS; ++q) red[wave][q][lane] = sum[q];
    __syncthreads();
    double sq = 0.0;
    for (int t = threadIdx.x; t < 64 * NS; t += 512) {
        const int q = t >> 6, jl = t & 63, j = 64 * q + jl;
        if (j < d) {
            unsigned long long tot = 0ull;
#pragma unroll
            for (int w = 0; w < 8; ++w) tot += red[w][q][jl];
            const float mean = (float)(((double)(long long)tot * (1.0 / 4294967296.0)) / (double)cnt);
            write_centroid(run, c, d, j, mean);
            sq += (double)mean * (double)mean;
        }
    }
    write_norm(run, c, sq, norm_sh);
}

// grid: (clusters, ranges).  Ranges are cut where the assignments are aligned to four of them; the first one also
// takes what comes before.  ONE: a single range, the centroid is written here; otherwise the range's sums go to
// part[cluster][range][d] and its number of members to order[cluster][range].
// What bounds it is the largest cluster of a range (early assignments are lopsided), hence eight wavefronts, eight rows in
// flight each; little LDS (indices as 16-bit distances, the sums in their place afterwards), as the k-means runs
// of a build and its other kernels share the compute units.
constexpr int KM_THREADS = 512, KM_WAVES = KM_THREADS / 64;

template <int NS, bool ONE>
__global__ __launch_bounds__(KM_THREADS) void kmeans_members_kernel(const float *__restrict__ Z, long long N, int d, KmRuns R)
{
    const KmRun &run = R.run[blockIdx.z];
    if ((int)blockIdx.x >= run.k) return;
    const int32_t *__restrict__ assign = run.assign;
    unsigned long long *__restrict__ part = run.part;
    constexpr int LIST_BYTES = 2 * (KM_RANGE + 4), RED_BYTES = 8 * (KM_WAVES / 2) * NS * 64;
    __shared__ __align__(16) unsigned char room[LIST_BYTES > RED_BYTES ? LIST_BYTES : RED_BYTES];
    unsigned short *members = (unsigned short *)room;   // distances from the range's start
    unsigned long long(*red)[NS][64] = (unsigned long long(*)[NS][64])room;   // [KM_WAVES / 2], once the rows are added up
    __shared__ double norm_sh[KM_WAVES];
    __shared__ int found;
    const int c = blockIdx.x, lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (threadIdx.x == 0) {
        found = 0;
        if (ONE && c == 0 && !run.keep_counts) {
            run.nflagged[0] = 0;
            run.nflagged[1] = 0;
        }
    }
    __syncthreads();
    const int head = (int)((16 - ((uintptr_t)assign & 15)) & 15) / 4;   // until the next multiple of 16 bytes
    const long long lo = (long long)blockIdx.y * KM_RANGE + head;       // where the range's whole groups of four begin
    const long long start = blockIdx.y == 0 ? 0 : lo;
    auto keep = [&](long long i) { members[atomicAdd(&found, 1)] = (unsigned short)(i - start); };
    if (blockIdx.y == 0 && (int)threadIdx.x < head && threadIdx.x < N && assign[threadIdx.x] == c) keep(threadIdx.x);
    {   // all loads requested before the first is looked at (a group past the end: the last whole one again, not
        // looked at)
        const long long whole = N - head > 3 ? (N - head) / 4 * 4 + head : head;   // end of the whole groups
        constexpr int PER = KM_RANGE / (4 * KM_THREADS);
        if (whole > head) {
            int4 v[PER];
#pragma unroll
            for (int u = 0; u < PER; ++u) {
                const long long i = lo + 4 * (KM_THREADS * u + (int)threadIdx.x);
                v[u] = *(const int4 *)(assign + (i < whole ? i : whole - 4));
            }
#pragma unroll
            for (int u = 0; u < PER; ++u) {
                const long long i = lo + 4 * (KM_THREADS * u + (int)threadIdx.x);
                const bool x = v[u].x == c, y = v[u].y == c, z = v[u].z == c, w = v[u].w == c;
                if ((x || y || z || w) && i < whole) {
                    if (x) keep(i);
                    if (y) keep(i + 1);
                    if (z) keep(i + 2);
                    if (w) keep(i + 3);
                }
            }
        }
        const long long i = whole + threadIdx.x;   // up to three left over
        if (threadIdx.x < 3 && i < N && i >= lo && i < lo + KM_RANGE && assign[i] == c) keep(i);
    }
    __syncthreads();
    const int cnt = found;
    unsigned long long sum[NS];
    int jc[NS];
#pragma unroll
    for (int q = 0; q < NS; ++q) {
        sum[q] = 0ull;
        jc[q] = 64 * q + lane < d ? 64 * q + lane : d - 1;
    }
    int held = 0;
    // eight rows at a time per wavefront, all loads unconditional (see kmeans_partial_kernel for the arithmetic)
    for (int u0 = 8 * wave; u0 < cnt; u0 += 8 * KM_WAVES) {
        float z[8][NS];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int row = __builtin_amdgcn_readfirstlane((int)start + members[u0 + u < cnt ? u0 + u : cnt - 1]);
            const float *__restrict__ zrow = Z + (long long)row * d;
#pragma unroll
            for (int q = 0; q < NS; ++q) z[u][q] = zrow[jc[q]];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (u0 + u < cnt) {   // the same in every lane
                ++held;
#pragma unroll
                for (int q = 0; q < NS; ++q)
                    sum[q] += (unsigned long long)__double_as_longlong(fma((double)z[u][q], 4294967296.0, 6755399441055744.0));
            }
    }
    __syncthreads();   // the list has been read
    if (wave >= KM_WAVES / 2)
#pragma unroll
        for (int q = 0; q < NS; ++q) red[wave - KM_WAVES / 2][q][lane] = sum[q] - (unsigned long long)held * FIX_MAGIC_BITS;
    __syncthreads();
    if (wave < KM_WAVES / 2)
#pragma unroll
        for (int q = 0; q < NS; ++q) red[wave][q][lane] += sum[q] - (unsigned long long)held * FIX_MAGIC_BITS;
    __syncthreads();
    if (ONE && cnt == 0) return;   // an empty cluster keeps its centroid (the same in every thread)
    double sq = 0.0;
    for (int t = threadIdx.x; t < 64 * NS; t += KM_THREADS) {
        const int q = t >> 6, jl = t & 63, j = 64 * q + jl;
        if (j < d) {
            unsigned long long tot = 0ull;
#pragma unroll
            for (int w = 0; w < KM_WAVES / 2; ++w) tot += red[w][q][jl];
            if (ONE) {
                const float mean = (float)(((double)(long long)tot * (1.0 / 4294967296.0)) / (double)cnt);
                write_centroid(run, c, d, j, mean);
                sq += (double)mean * (double)mean;
            } else {
                part[((size_t)c * gridDim.y + blockIdx.y) * (size_t)d + j] = tot;
            }
        }
    }
    if (ONE)
        write_norm(run, c, sq, norm_sh);
    else if (threadIdx.x == 0)
        run.order[c * gridDim.y + blockIdx.y] = cnt;
}

// Adds up a cluster's ranges and writes its centroid; one workgroup per cluster.
__global__ __launch_bounds__(256) void kmeans_ranges_kernel(int d, int ranges, KmRuns R)
{
    const KmRun &run = R.run[blockIdx.y];
    if ((int)blockIdx.x >= run.k) return;
    const unsigned long long *__restrict__ part = run.part;
    const int *__restrict__ cnts = run.order;
    __shared__ double norm_sh[4];
    const int c = blockIdx.x;
    if (threadIdx.x == 0 && c == 0 && !run.keep_counts) {
        run.nflagged[0] = 0;
        run.nflagged[1] = 0;
    }
    int cnt = 0;
    for (int r = 0; r < ranges; ++r) cnt += cnts[c * ranges + r];
    if (cnt == 0) return;  // an empty cluster keeps its centroid (the same in every thread)
    double sq = 0.0;
    for (int j = threadIdx.x; j < d; j += 256) {
        unsigned long long tot = 0ull;
#pragma unroll 8
        for (int r = 0; r < ranges; ++r) tot += part[((size_t)c * ranges + r) * (size_t)d + j];
        const float mean = (float)(((double)(long long)tot * (1.0 / 4294967296.0)) / (double)cnt);
        write_centroid(run, c, d, j, mean);
        sq += (double)mean * (double)mean;
    }
    write_norm(run, c, sq, norm_sh);
}

template <int NS>
static void launch_members(const float *Z, long long N, int d, const KmRuns &runs, int kmax, hipStream_t s)
{
    const int ranges = kmeans_ranges(N);
    const dim3 grid((unsigned)kmax, (unsigned)ranges, (unsigned)runs.count);
    if (ranges == 1) {
        hipLaunchKernelGGL((kmeans_members_kernel<NS, true>), grid, dim3(KM_THREADS), 0, s, Z, N, d, runs);
    } else {
        hipLaunchKernelGGL((kmeans_members_kernel<NS, false>), grid, dim3(KM_THREADS), 0, s, Z, N, d, runs);
        hipLaunchKernelGGL(kmeans_ranges_kernel, dim3((unsigned)kmax, (unsigned)runs.count), dim3(256), 0, s, d, ranges, runs);
    }
}

hipError_t launch_kmeans_update(const float *Z, long long N, int d, const KmRuns &runs, int parity, hipStream_t s)
{
    const int ns = (d + 63) / 64;
    int k = 0;
    for (int q = 0; q < runs.count; ++q) k = runs.run[q].k > k ? runs.run[q].k : k;
    if (runs.by_members) {
        switch (ns) {
            case 1: launch_members<1>(Z, N, d, runs, k, s); break;
            case 2: launch_members<2>(Z, N, d, runs, k, s); break;
            case 3: launch_members<3>(Z, N, d, runs, k, s); break;
            case 4: launch_members<4>(Z, N, d, runs, k, s); break;
            case 5: launch_members<5>(Z, N, d, runs, k, s); break;
            case 6: launch_members<6>(Z, N, d, runs, k, s); break;
            case 7: launch_members<7>(Z, N, d, runs, k, s); break;
            default: launch_members<8>(Z, N, d, runs, k, s); break;
        }
        return hipGetLastError();
    }
    if (runs.count != 1) return hipErrorInvalidValue;
    const KmRun &r = runs.run[0];
    int *counts = r.counts2 + (size_t)(parity & 1) * k, *counts_next = r.counts2 + (size_t)((parity + 1) & 1) * k;
    int *cursor = r.cursor2 + (size_t)(parity & 1) * k, *cursor_next = r.cursor2 + (size_t)((parity + 1) & 1) * k;
    const unsigned blocks = (unsigned)((N + KM_POINTS - 1) / KM_POINTS);
    hipLaunchKernelGGL(kmeans_count_kernel, dim3(blocks), dim3(256), sizeof(int) * (size_t)k, s, r.assign, N, k, counts);
    hipLaunchKernelGGL(kmeans_scatter_kernel, dim3(blocks), dim3(256), 2 * sizeof(int) * (size_t)k, s, r.assign, N, k,
                       counts, cursor, r.order, r.offs);
    if (ns <= 8) {
        const int M = kmeans_sum_chunk(N);
        const unsigned pblocks = (unsigned)(((N + M - 1) / M + 3) / 4);
#define LCN_SUM_PARTIAL(NS_)                                                                                       \
    hipLaunchKernelGGL((kmeans_partial_kernel<NS_>), dim3(pblocks), dim3(256), 0, s, Z, N, d, M, r.assign, r.order,   \
                       r.part);                                                                                        \
    hipLaunchKernelGGL((kmeans_mean_kernel<NS_>), dim3((unsigned)k), dim3(512), 0, s, r.part, d, M, counts,            \
                       counts_next, cursor_next, r)
        switch (ns) {
            case 1: LCN_SUM_PARTIAL(1); break;
            case 2: LCN_SUM_PARTIAL(2); break;
            case 3: LCN_SUM_PARTIAL(3); break;
            case 4: LCN_SUM_PARTIAL(4); break;
            case 5: LCN_SUM_PARTIAL(5); break;
            case 6: LCN_SUM_PARTIAL(6); break;
            case 7: LCN_SUM_PARTIAL(7); break;
            default: LCN_SUM_PARTIAL(8); break;
        }
#undef LCN_SUM_PARTIAL
        return hipGetLastError();
    }
    int *reset = r.keep_counts ? nullptr : r.nflagged;
    if ((long long)k * ((d + 63) / 64) >= 512)
        hipLaunchKernelGGL((kmeans_sum_kernel<64, 16>), dim3((unsigned)k, (unsigned)((d + 63) / 64)), dim3(1024), 0, s, Z,
                           d, k, counts, r.offs, r.order, r.cent, counts_next, cursor_next, reset);
    else   // few clusters: narrower slices, four times the workgroups
        hipLaunchKernelGGL((kmeans_sum_kernel<16, 16>), dim3((unsigned)k, (unsigned)((d + 15) / 16)), dim3(1024), 0, s, Z,
                           d, k, counts, r.offs, r.order, r.cent, counts_next, cursor_next, reset);
    hipError_t e = hipGetLastError();
    // a centroid's slices are written by several workgroups: the planes and norms follow in a launch of their own
    if (e == hipSuccess && r.first && reset) {   // (the last iteration's are not used)
        KmRuns again = runs;
        again.run[0].pick = nullptr;
        e = launch_kmeans_start(nullptr, d, again, s);
    }
    return e;
}

// ------------------------------------------------------------ bucket sort --
//
// Stable counting sort of the point indices of each side (X, Y) by bucket,
// per hash round.  Chunks of CH consecutive indices are histogrammed, the
// histograms are prefixed over chunks and buckets, and each chunk is then
// scattered by one wavefront that ranks equal keys in index order.

constexpr int CH = 1024;

__global__ void scan_i64_kernel(long long *data, long long n, long long *data2, long long n2);

// Inclusive scan over the lanes of a wavefront.
template <class T>
__device__ inline T wave_inclusive_scan(T v)
{
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const T up = __shfl_up(v, o, 64);
        if (lane >= o) v += up;
    }
    return v;
}

// Exclusive scan of per-thread values across a workgroup of WAVES wavefronts: returns the sum of the values of all lower threads;
// *total receives the sum of all.  wsum: WAVES words of LDS that no scan since the last but one has used.
template <int WAVES, class T>
__device__ inline T block_exclusive_scan(T local, T *wsum, T *total)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const T incl = wave_inclusive_scan(local);
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    T before = 0, all = 0;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
        const T v = wsum[w];
        if (w < wave) before += v;
        all += v;
    }
    *total = all;
    return before + incl - local;
}

int sort_chunks(long long n, long long m)
{
    long long mx = n > m ? n : m;
    return (int)((mx + CH - 1) / CH);
}

__device__ inline long long side_count(const SortBuffers &B, int side) { return side == 0 ? B.n : B.m; }

// grid: (chunks, R, 2)
__global__ __launch_bounds__(256) void sort_hist_kernel(SortBuffers B)
{
    extern __shared__ int hist[];
    const int chunk = blockIdx.x, r = blockIdx.y, side = blockIdx.z;
    const long long cnt = side_count(B, side);
    for (int t = threadIdx.x; t < B.b; t += blockDim.x) hist[t] = 0;
    __syncthreads();
    const long long base = (long long)chunk * CH;
    const int32_t *bk = B.bucket + (long long)r * (B.n + B.m) + (side ? B.n : 0);
    for (int t = threadIdx.x; t < CH; t += blockDim.x) {
        long long i = base + t;
        if (i < cnt) atomicAdd(&hist[bk[i]], 1);
    }
    __syncthreads();
    int *dst = B.hist + (((long long)side * B.R + r) * B.chunks + chunk) * B.b;
    for (int t = threadIdx.x; t < B.b; t += blockDim.x) dst[t] = hist[t];
}

// one thread per (side, round, bucket): exclusive prefix over chunks, bucket totals
__global__ void sort_chunk_prefix_kernel(SortBuffers B)
{
    int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= 2 * B.R * B.b) return;
    int beta = t % B.b;
    int sr = t / B.b;  // side * R + r
    int *h = B.hist + (long long)sr * B.chunks * B.b + beta;
    int run = 0;
    for (int c = 0; c < B.chunks; c += 8) {   // eight loads at a time
        int v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = h[(long long)(c + u < B.chunks ? c + u : B.chunks - 1) * B.b];
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (c + u < B.chunks) {
                h[(long long)(c + u) * B.b] = run;
                run += v[u];
            }
    }
    B.totals[t] = run;
}

// Single workgroup: bucket offsets per (side, round), a wavefront for each; tile offsets over all blocks; totals.
// What bounds it is the chain of its steps, so it has few barriers: three rounds of 128 buckets 4.8 us
// (17 with a scan by all of 1024 threads per side and round, and the maxima by atomics).
__global__ __launch_bounds__(256) void sort_offsets_kernel(SortBuffers B)
{
    __shared__ int wsum[2][4];
    __shared__ long long sums[3][4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    for (int sr = wave; sr < 2 * B.R; sr += 4) {
        const int *tot = B.totals + sr * B.b;
        int *off = B.off + sr * (B.b + 1);
        int carry = 0;
        for (int t0 = 0; t0 < B.b; t0 += 256) {
            const int i0 = t0 + 4 * lane;
            int v[4], sum = 0;
#pragma unroll
            for (int q = 0; q < 4; ++q) sum += v[q] = i0 + q < B.b ? tot[i0 + q] : 0;
            const int incl = wave_inclusive_scan(sum);
            int run = carry + incl - sum;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if (i0 + q < B.b) off[i0 + q] = run;
                run += v[q];
            }
            carry += __shfl(incl, 63, 64);
        }
        if (lane == 0) off[B.b] = carry;
    }
    // blocks in (round, bucket) order: values (nx * ny), 64 x 64 build tiles, the largest ones
    const int nb = B.R * B.b;
    long long pairs = 0, bytes = 0, side = 0;
    int carry = 0;
    for (int t0 = 0, turn = 0; t0 < nb; t0 += 1024, turn ^= 1) {
        const int i0 = t0 + 4 * tid;
        int tiles[4], sum = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const bool in = i0 + q < nb;
            const int nx = in ? B.totals[i0 + q] : 0, ny = in ? B.totals[nb + i0 + q] : 0;
            pairs += (long long)nx * ny;
            if (in) bytes = max(bytes, bucket_block_bytes(nx, ny));
            side = max(side, (long long)max(nx, ny));
            sum += tiles[q] = (int)(((nx + 63ll) / 64) * ((ny + 63ll) / 64));
        }
        int all;
        int run = carry + block_exclusive_scan<4>(sum, wsum[turn], &all);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if (i0 + q < nb) B.tile_off[i0 + q] = run;
            run += tiles[q];
        }
        carry += all;
    }
    for (int o = 32; o > 0; o >>= 1) {
        pairs += __shfl_xor(pairs, o, 64);
        bytes = max(bytes, __shfl_xor(bytes, o, 64));
        side = max(side, __shfl_xor(side, o, 64));
    }
    if (lane == 0) sums[0][wave] = pairs, sums[1][wave] = bytes, sums[2][wave] = side;
    __syncthreads();
    if (tid == 0) {
        for (int w = 1; w < 4; ++w) {
            pairs += sums[0][w];
            bytes = max(bytes, sums[1][w]);
            side = max(side, sums[2][w]);
        }
        B.tile_off[nb] = carry;
        B.totals_out[0] = pairs;
        B.totals_out[1] = carry;
        B.totals_out[2] = bytes;
        B.totals_out[3] = side;
    }
}

// grid: (chunks, R, 2); one workgroup of 16 wavefronts per chunk of 1024 elements, one element
// per thread.  Stable: a wavefront ranks its 64 elements among equal keys by ballots, then the
// wavefronts take their places in the running bucket positions one after the other (128 buckets: 4.9 us; 13.2 with the ballots
// a distinct key after the other).
__global__ __launch_bounds__(1024) void sort_scatter_kernel(SortBuffers B)
{
    extern __shared__ int running[];
    const int chunk = blockIdx.x, r = blockIdx.y, side = blockIdx.z;
    const long long cnt = side_count(B, side);
    const long long base = (long long)chunk * CH;
    if (base >= cnt) return;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int sr = side * B.R + r;
    const int *pre = B.hist + ((long long)sr * B.chunks + chunk) * B.b;
    const int *off = B.off + sr * (B.b + 1);
    for (int t = threadIdx.x; t < B.b; t += 1024) running[t] = off[t] + pre[t];
    const int32_t *bk = B.bucket + (long long)r * (B.n + B.m) + (side ? B.n : 0);
    int *perm = B.perm + (side ? (long long)B.R * B.n + (long long)r * B.m : (long long)r * B.n);
    int *pos = B.pos + (side ? (long long)B.R * B.n + (long long)r * B.m : (long long)r * B.n);
    const long long i = base + threadIdx.x;
    const bool valid = i < cnt;
    const int key = valid ? bk[i] : -1;
    // rank of this lane among the lanes of its wavefront with the same key (lower lanes first): those whose keys agree in
    // every bit
    unsigned long long same = __ballot(valid);
    for (int bit = 1; bit < B.b; bit <<= 1) {
        const unsigned long long set = __ballot(valid && (key & bit));
        same &= key & bit ? set : ~set;
    }
    const int rank = __popcll(same & ((1ull << lane) - 1ull)), group = __popcll(same);
    int dst = 0;
    for (int w = 0; w < CH / 64; ++w) {
        __syncthreads();   // running[] as the wavefronts before w left it (w = 0: as initialised)
        if (w == wave && valid) dst = running[key] + rank;
        __syncthreads();   // every lane of wavefront w has read before one lane per key moves the position on
        if (w == wave && valid && rank == group - 1) running[key] += group;
    }
    if (valid) {
        perm[dst] = (int)i;
        pos[i] = dst;
    }
}

// per (round, row): the slice of the other side's bucket-ordered vector the row
// multiplies; per row: the length of its record (written to rowbase, scanned after)
__global__ void seg_kernel(SortBuffers B)
{
    const int side = blockIdx.y;
    const long long cnt = side_count(B, side);
    long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= cnt) return;
    const long long other = side ? B.n : B.m;
    long long total = 0;
    for (int r = 0; r < B.R; ++r) {
        const int32_t *bk = B.bucket + (long long)r * (B.n + B.m) + (side ? B.n : 0);
        const int beta = bk[i];
        const int *off_ot = B.off + ((1 - side) * B.R + r) * (B.b + 1);
        Seg sg;
        sg.len = off_ot[beta + 1] - off_ot[beta];
        sg.vstart = (int)((long long)r * other + off_ot[beta]);
        (side ? B.seg_y : B.seg_x)[(long long)r * cnt + i] = sg;
        total += sg.len;
    }
    (side ? B.rowbase_y : B.rowbase_x)[i] = total;
}

hipError_t launch_bucket_sort(const SortBuffers &B, hipStream_t s)
{
    dim3 grid(B.chunks, B.R, 2);
    size_t lds = sizeof(int) * (size_t)B.b;
    hipLaunchKernelGGL(sort_hist_kernel, grid, dim3(256), lds, s, B);
    int t = 2 * B.R * B.b;
    hipLaunchKernelGGL(sort_chunk_prefix_kernel, dim3((t + 127) / 128), dim3(128), 0, s, B);
    hipLaunchKernelGGL(sort_offsets_kernel, dim3(1), dim3(256), 0, s, B);
    hipLaunchKernelGGL(sort_scatter_kernel, grid, dim3(1024), lds, s, B);
    long long mx = B.n > B.m ? B.n : B.m;
    hipLaunchKernelGGL(seg_kernel, dim3((unsigned)((mx + 255) / 256), 2), dim3(256), 0, s, B);
    hipLaunchKernelGGL(scan_i64_kernel, dim3(2), dim3(1024), 0, s, B.rowbase_x, B.n, B.rowbase_y, B.m);
    return hipGetLastError();
}

// Packed per-row metadata read by the sweeps, one record per row:
//   [0:1] start of the row's record of sparse values (int64)
//   [2]   marginal (float)          [4:5] its natural log (double)
//   [6 + 2r], [7 + 2r]  round r: what takes an entry's number in the record to its place in the other side's
//                       bucket-ordered vector (modulo 2^32), and the number of the first entry past the round
//   [6 + 2R + r]        round r: position of the row in its own side's bucket order
int meta_stride_for(int R) { return (6 + 3 * R + 3) / 4 * 4; }

__global__ void meta_kernel(SortBuffers B, const float *a, const float *b)
{
    const int side = blockIdx.y;
    const long long cnt = side_count(B, side);
    long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= cnt) return;
    int *rec = (side ? B.meta_y : B.meta_x) + i * B.meta_stride;
    const long long base = B.R > 0 ? (side ? B.rowbase_y : B.rowbase_x)[i] : 0;
    const float marg = (side ? b : a)[i];
    const double lm = log((double)marg);
    rec[0] = (int)(unsigned)(base & 0xffffffffll);
    rec[1] = (int)(base >> 32);
    rec[2] = __float_as_int(marg);
    rec[3] = 0;
    rec[4] = __double2loint(lm);
    rec[5] = __double2hiint(lm);
    const int *pos = B.pos + (side ? (long long)B.R * B.n : 0);
    int at = 0;
    for (int r = 0; r < B.R; ++r) {
        const Seg sg = (side ? B.seg_y : B.seg_x)[(long long)r * cnt + i];
        rec[6 + 2 * r] = (int)((unsigned)sg.vstart - (unsigned)at);
        at += sg.len;
        rec[7 + 2 * r] = at;
        rec[6 + 2 * B.R + r] = pos[(long long)r * cnt + i];
    }
}

hipError_t launch_build_meta(const SortBuffers &B, const float *a, const float *b, hipStream_t s)
{
    long long mx = B.n > B.m ? B.n : B.m;
    hipLaunchKernelGGL(meta_kernel, dim3((unsigned)((mx + 255) / 256), 2), dim3(256), 0, s, B, a, b);
    return hipGetLastError();
}

// ------------------------------------------------------------- CSR export --
//
// Row i of the pattern is the union over rounds of the Y members of the
// bucket x_i fell into; a pair that an earlier round already holds is
// skipped.  Members of a bucket are in ascending index order (stable sort),
// so the union is an R-way merge of ascending lists.

__device__ inline bool owned_by_earlier_round(const int32_t *bucket, long long N, long long n, int r, long long i,
                                              int j)
{
    for (int q = 0; q < r; ++q)
        if (bucket[(long long)q * N + i] == bucket[(long long)q * N + n + j]) return true;
    return false;
}

// One row by one thread: the R-way merge written out.  Used for rows too long for the
// wavefront version below.
template <bool FILL>
__device__ inline void csr_row_serial(const SortBuffers &B, long long i, const float *vals, const float *vals2,
                                      int log_values, long long *rowcount, const long long *rowptr, int32_t *colidx,
                                      float *val, float *val2)
{
    const long long N = B.n + B.m;
    int head[8], segstart[8];
    int run = 0;
    for (int r = 0; r < B.R; ++r) {
        head[r] = 0;
        segstart[r] = run;
        run += B.seg_x[(long long)r * B.n + i].len;
    }
    const long long base = B.rowbase_x[i];
    long long outp = FILL ? rowptr[i] : 0;
    long long cnt = 0;
    while (true) {
        int bestj = 0x7fffffff, bestr = -1;
        for (int r = 0; r < B.R; ++r) {
            const Seg sg = B.seg_x[(long long)r * B.n + i];
            const int *yperm = B.perm + (long long)B.R * B.n + (long long)r * B.m;
            const int seg0 = sg.vstart - (int)((long long)r * B.m);
            // skip entries an earlier round owns
            while (head[r] < sg.len &&
                   owned_by_earlier_round(B.bucket, N, B.n, r, i, yperm[seg0 + head[r]]))
                ++head[r];
            if (head[r] < sg.len) {
                int j = yperm[seg0 + head[r]];
                if (j < bestj) {
                    bestj = j;
                    bestr = r;
                }
            }
        }
        if (bestr < 0) break;
        if (FILL) {
            if (colidx) colidx[outp] = bestj;
            const long long at = base + segstart[bestr] + head[bestr];
            if (val) val[outp] = log_values ? expf(vals[at]) : vals[at];
            if (val2) val2[outp] = vals2[at];
            ++outp;
        }
        ++cnt;
        ++head[bestr];
    }
    if (!FILL) rowcount[i] = cnt;
}

// One wavefront per row.  The row's stored columns (all rounds, T of them) go into LDS, a dropped
// pair as INT_MAX; the place of a kept pair in the row is the number of kept columns below its own,
// counted by brute force over the T entries (T^2 / 64 LDS reads per lane, T ~ 100).  With one round
// the record already is the CSR row.  FILL = false only counts the kept pairs.
constexpr int CSR_ROW_MAX = 2048;  // entries of a row the wavefront version holds

template <bool FILL>
__global__ __launch_bounds__(256) void csr_kernel(SortBuffers B, const float *vals, const float *vals2,
                                                  int log_values, long long *rowcount, const long long *rowptr,
                                                  int32_t *colidx, float *val, float *val2)
{
    __shared__ int cols_sh[4][CSR_ROW_MAX];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const long long i = (long long)blockIdx.x * 4 + w;
    const bool live = i < B.n;
    const long long N = B.n + B.m;
    int T = 0;
    if (live)
        for (int r = 0; r < B.R; ++r) T += B.seg_x[(long long)r * B.n + i].len;
    const long long base = live ? B.rowbase_x[i] : 0;
    const bool serial = live && B.R > 1 && T > CSR_ROW_MAX;
    const bool wide = live && B.R > 1 && !serial;
    int *cols = cols_sh[w];
    if (wide) {
        int off = 0;
        for (int r = 0; r < B.R; ++r) {
            const Seg sg = B.seg_x[(long long)r * B.n + i];
            const int *yperm = B.perm + (long long)B.R * B.n + (long long)r * B.m;
            const int seg0 = sg.vstart - (int)((long long)r * B.m);
            for (int e = lane; e < sg.len; e += 64) {
                const int j = yperm[seg0 + e];
                cols[off + e] = owned_by_earlier_round(B.bucket, N, B.n, r, i, j) ? 0x7fffffff : j;
            }
            off += sg.len;
        }
    }
    __syncthreads();
    if (!live) return;
    if (serial) {
        if (lane == 0) csr_row_serial<FILL>(B, i, vals, vals2, log_values, rowcount, rowptr, colidx, val, val2);
        return;
    }
    const long long outp = FILL ? rowptr[i] : 0;
    long long kept = 0;
    for (int t0 = 0; t0 < T; t0 += 64) {
        const int t = t0 + lane;
        int j = 0x7fffffff;
        if (t < T) j = B.R > 1 ? cols[t] : B.perm[(long long)B.R * B.n + B.seg_x[i].vstart + t];
        const bool keep = j != 0x7fffffff;
        if (!FILL) {
            kept += __popcll(__ballot(keep));
            continue;
        }
        if (!keep) continue;
        int rank = t;  // one round: the record is in column order and nothing is dropped
        if (B.R > 1) {
            rank = 0;
#pragma unroll 8
            for (int q = 0; q < T; ++q) rank += cols[q] < j ? 1 : 0;
        }
        if (colidx) colidx[outp + rank] = j;
        if (val) val[outp + rank] = log_values ? expf(vals[base + t]) : vals[base + t];
        if (val2) val2[outp + rank] = vals2[base + t];
    }
    if (!FILL && lane == 0) rowcount[i] = kept;
}

hipError_t launch_csr_count(const Handle &h, long long *rowcount, hipStream_t s)
{
    hipLaunchKernelGGL(csr_kernel<false>, dim3((unsigned)((h.n + 3) / 4)), dim3(256), 0, s, h.sort, h.vals_x,
                       (const float *)nullptr, h.log_domain, rowcount, (const long long *)nullptr, (int32_t *)nullptr,
                       (float *)nullptr, (float *)nullptr);
    return hipGetLastError();
}

hipError_t launch_csr_fill(const Handle &h, const long long *rowptr, int32_t *colidx, float *val, hipStream_t s)
{
    hipLaunchKernelGGL(csr_kernel<true>, dim3((unsigned)((h.n + 3) / 4)), dim3(256), 0, s, h.sort, h.vals_x,
                       (const float *)nullptr, h.log_domain, (long long *)nullptr, rowptr, colidx, val,
                       (float *)nullptr);
    return hipGetLastError();
}

// exp(t) for a result in single precision: 2^k e^r with the Taylor polynomial of degree 9 on |r| <= ln(2) / 2 (remainder
// below 7e-12, against 6e-8 of the rounding: rounded to single precision 8 results in a million differ from the library's);
// minus infinity and what is not a number give zero.  The two parts of ln 2 are those of fdlibm's exp (the upper one has
// 32 bits, so that k times it is exact).
__device__ inline float exp_to_float(double t)
{
    t = fmin(fmax(t, -200.0), 200.0);
    const double k = rint(t * 1.4426950408889634074);
    const double r = fma(-k, 1.9082149292705877e-10, fma(-k, 0.693147180369123816490, t));
    double p = 1.0 / 362880.0;
    p = fma(p, r, 1.0 / 40320.0);
    p = fma(p, r, 1.0 / 5040.0);
    p = fma(p, r, 1.0 / 720.0);
    p = fma(p, r, 1.0 / 120.0);
    p = fma(p, r, 1.0 / 24.0);
    p = fma(p, r, 1.0 / 6.0);
    p = fma(p, r, 0.5);
    p = fma(p, r, 1.0);
    p = fma(p, r, 1.0);
    return (float)ldexp(p, (int)k);
}

// The plan's rows of the dense kernel (one bucket: every record holds all columns in their order, every entry of the
// block is written).  A wavefront takes four rows and 1024 columns: a column's scaling is read once for four rows, and a
// block of few rows still gives every unit work.  What bounds it is memory (0.8 GB at 10 000 x 10 000: 182
// us; a row per wavefront, the library's exp and a clear before it: 443 + 82 us; all columns per wavefront: 341 us, too
// few in flight).
constexpr int PLAN_ROWS = 4, PLAN_COLS = 1024;
__global__ __launch_bounds__(256) void plan_dense_kernel(const long long *__restrict__ rowbase,
                                                         const float *__restrict__ vals, long long m, long long i0,
                                                         long long nrows, const double *__restrict__ log_u,
                                                         const double *__restrict__ log_v, float *__restrict__ out)
{
    const int lane = threadIdx.x & 63;
    const long long parts = (m + PLAN_COLS - 1) / PLAN_COLS;
    const long long w = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
    const long long l0 = w / parts * PLAN_ROWS, j0 = w % parts * PLAN_COLS;
    if (l0 >= nrows) return;
    const long long j1 = j0 + PLAN_COLS < m ? j0 + PLAN_COLS : m;
    const float *row[PLAN_ROWS];
    double u[PLAN_ROWS];
#pragma unroll
    for (int q = 0; q < PLAN_ROWS; ++q) {   // past the last row: the last one again, not written
        const long long i = i0 + (l0 + q < nrows ? l0 + q : nrows - 1);
        row[q] = vals + rowbase[i];
        u[q] = log_u[i];
    }
    for (long long j = j0 + lane; j < j1; j += 64) {
        const double v = log_v[j];
        float k[PLAN_ROWS];
#pragma unroll
        for (int q = 0; q < PLAN_ROWS; ++q) k[q] = row[q][j];
#pragma unroll
        for (int q = 0; q < PLAN_ROWS; ++q)
            if (l0 + q < nrows) out[(l0 + q) * m + j] = exp_to_float((double)k[q] + u[q] + v);
    }
}

// Sparse part of the plan for a block of rows, one wavefront per row: every stored pair of the
// row that no earlier round owns adds u_i val_ij v_j to out[i - i0][j] (values held as logs:
// sets exp(log u_i + val_ij + log v_j)).  Each (i, j) is touched by one lane only.
__global__ __launch_bounds__(256) void plan_sparse_kernel(SortBuffers B, const float *__restrict__ vals_x,
                                                          int log_values, long long i0, long long nrows,
                                                          const double *__restrict__ lin_u,
                                                          const double *__restrict__ lin_v,
                                                          const double *__restrict__ acc_y,
                                                          const double *__restrict__ acc_z, int lp,
                                                          float *__restrict__ out)
{
    const long long li = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (li >= nrows) return;
    const long long i = i0 + li;
    const int lane = threadIdx.x & 63;
    const long long N = B.n + B.m;
    const double ui = lin_u[i];
    const double scale = log_values ? 0.0 : exp(acc_y[lp] + acc_z[lp]);
    long long at = B.rowbase_x[i];
    for (int r = 0; r < B.R; ++r) {
        const Seg sg = B.seg_x[(long long)r * B.n + i];
        const int *yperm = B.perm + (long long)B.R * B.n + (long long)r * B.m;
        const int seg0 = sg.vstart - (int)((long long)r * B.m);
        for (int e = lane; e < sg.len; e += 64) {
            const int j = yperm[seg0 + e];
            if (owned_by_earlier_round(B.bucket, N, B.n, r, i, j)) continue;
            const double v = (double)vals_x[at + e];
            float *dst = out + li * B.m + j;
            if (log_values) {
                *dst = exp_to_float(v + ui + lin_v[j]);
            } else {
                *dst += (float)(v * ui * lin_v[j] * scale);
            }
        }
        at += sg.len;
    }
}

hipError_t launch_plan_sparse(const Handle &h, long long i0, long long nrows, float *out, hipStream_t s)
{
    const long long waves = (nrows + PLAN_ROWS - 1) / PLAN_ROWS * ((h.m + PLAN_COLS - 1) / PLAN_COLS);
    if (h.mode == LCN_MODE_DENSE)
        hipLaunchKernelGGL(plan_dense_kernel, dim3((unsigned)((waves + 3) / 4)), dim3(256), 0, s, h.sort.rowbase_x, h.vals_x, h.m,
                           i0, nrows, h.lin_u, h.lin_v, out);
    else
        hipLaunchKernelGGL(plan_sparse_kernel, dim3((unsigned)((nrows + 3) / 4)), dim3(256), 0, s, h.sort, h.vals_x,
                           h.log_domain, i0, nrows, h.lin_u, h.lin_v, h.acc[0], h.acc[1], h.lp, out);
    return hipGetLastError();
}

// rec / rec2 (nullable): values in the layout of X's row records; val / val2: the same in CSR order
hipError_t launch_csr_values(const Handle &h, const float *rec, const float *rec2, const long long *rowptr, float *val,
                             float *val2, hipStream_t s)
{
    hipLaunchKernelGGL(csr_kernel<true>, dim3((unsigned)((h.n + 3) / 4)), dim3(256), 0, s, h.sort, rec, rec2, 0,
                       (long long *)nullptr, rowptr, (int32_t *)nullptr, val, val2);
    return hipGetLastError();
}

// in-place exclusive scan of n int64 values by one block; data[n] receives the total
// One workgroup; tiles of 4096 elements, four consecutive ones per thread, the next tile's loads under way while one is scanned
// (two sides of 20 000 elements: 12.1 us, 14.6 without).
__global__ __launch_bounds__(1024) void scan_i64_kernel(long long *data, long long n, long long *data2, long long n2)
{
    __shared__ long long wsum[2][16];
    if (blockIdx.x == 1) {
        data = data2;
        n = n2;
    }
    const int tid = threadIdx.x;
    long long carry = 0, v[4], next[4];
    auto load = [&](long long (&to)[4], long long i0) {   // past the end the last element, which is not used
#pragma unroll
        for (int q = 0; q < 4; ++q) to[q] = data[i0 + q < n ? i0 + q : n - 1];
    };
    if (n > 0) load(v, 4 * tid);
    int turn = 0;
    for (long long t0 = 0; t0 < n; t0 += 4096, turn ^= 1) {
        const long long i0 = t0 + 4 * tid;
        load(next, i0 + 4096);
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = i0 + q < n ? v[q] : 0;
        long long tile_total;
        long long run = carry + block_exclusive_scan<16>(v[0] + v[1] + v[2] + v[3], wsum[turn], &tile_total);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if (i0 + q < n) data[i0 + q] = run;
            run += v[q];
            v[q] = next[q];
        }
        carry += tile_total;
    }
    if (tid == 0) data[n] = carry;
}

hipError_t launch_scan_i64(long long *data, long long n, hipStream_t s)
{
    hipLaunchKernelGGL(scan_i64_kernel, dim3(1), dim3(1024), 0, s, data, n, (long long *)nullptr, 0ll);
    return hipGetLastError();
}

}  // namespace lcn
