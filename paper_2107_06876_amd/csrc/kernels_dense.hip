// One whole iteration of dense Sinkhorn from one read of the kernel matrix.
//
// A half-iteration by itself is bound by reading the n x m matrix (rows of K for u, rows of its transpose for v).
// With the new u_i at hand while row i is still in registers, the row's share of the sums over columns
// costs one multiply-add per entry: with shift_i = log a_i - log u_i (previous u), E_ij = exp(k_ij +
// log v_j - shift_i) and t_i = sum_j E_ij,
//     log u_i = log a_i - shift_i - log t_i,
//     sum_i exp(k_ij + log u_i) v_j = sum_i E_ij a_i / t_i =: s_j,     log v_j = log b_j + log v_j - log s_j,
// so there is no second exponential either.  What bounds it is the one read of the matrix.
//
// A workgroup (one per compute unit, 1024 threads) takes RG rows at a time, each thread C columns of them, the next
// RG rows' loads in flight meanwhile; log v_j and the column sums stay in registers for the whole launch.
// RG * C is at most 24 (8 and 16 for one and two pieces, 12 .. 18 with a row at a time): two sets of values and two
// per column fill the 128 registers a thread has (30 spills; eighteen pieces spill one outside the loop).  The prefetch
// is unconditional (past the end the last row again): behind a condition the compiler waits for all loads.  A group
// past the end is not worked on: with two groups at a time whatever their number, 4000 x 4000 (three) took 27.4 us per
// iteration instead of 23.1.
// Every other iteration goes through the rows from the last to the first, so that what the iteration before read last is
// still in the 256 MB cache in front of the memory: 10 000 x 10 000 76.5 -> 72 us.  (More is not to be had from that cache: it
// answers at 7.2 TB/s, memory at 6.1.  A bare read of 400 MB takes 69.2 us in one direction and 63.6 in alternating ones.)
// The column sums of the workgroups, in single precision over n / (number of workgroups) rows, are added in double
// precision by dense_columns_kernel, which finishes v.
// 10 000 x 10 000 (400 MB): 160 us per iteration with two reads, 80 us so (5.0 TB/s).
// Root mean square error of log u, log v against 64 bits (two reads): 10 000 x 10 000 after 400 iterations 2.7e-7, 0.7e-7
// (1.4e-6, 1.4e-6), 4000 x 9000 after 1000 4.8e-7, 4.7e-7, left by the first iteration (1.9e-6, 1.8e-6), 200 000 x 64 after
// 50 3.1e-7, 1.8e-7 (4.8e-6, 5.0e-6).
#include "iter_common.h"

namespace lcn {

constexpr int DI_THREADS = 1024;
constexpr int DI_WAVES = DI_THREADS / 64;
// A row's sum above the first bounds what its smallest terms lose in single precision (terms below 1e-38) after the
// division by the sum.  A row outside the range gets its log-sum-exp with running maxima and stays out of the
// workgroup's column sums, and dense_columns_kernel takes every column from the transpose.  That is the first
// iteration from new scalings at most, or one in which a scaling moves by four orders of magnitude.
constexpr double DI_ROW_MIN = 1e-4, DI_MAX = 1e30;
constexpr double DI_COLUMN_MIN = 1e-20;   // the same for a column's sum, which is of order one here

// Workgroup barrier that waits for LDS only: the loads of the next rows stay in flight.
__device__ inline void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// log of a positive finite double to 2e-11: 2 atanh((m - 1) / (m + 1)) for the mantissa in [sqrt(1/2), sqrt(2)).
__device__ inline double short_log(double x)
{
    double m = __builtin_amdgcn_frexp_mant(x);
    int e = __builtin_amdgcn_frexp_exp(x);
    if (m < 0.70710678118654752440) {
        m += m;
        --e;
    }
    const double z = (m - 1.0) * fast_rcp(m + 1.0), q = z * z;
    double p = 2.0 / 11;
    p = fma(p, q, 2.0 / 9);
    p = fma(p, q, 2.0 / 7);
    p = fma(p, q, 2.0 / 5);
    p = fma(p, q, 2.0 / 3);
    p = fma(p, q, 2.0);
    return fma((double)e, 0.69314718055994530942, p * z);
}

// Log-sum-exp of k[e] + p[e] over `len` entries by one wavefront's share (from `first`, every `step`), with a
// running maximum per lane; merged over the wavefront.
__device__ inline void wave_lse(const float *__restrict__ k, const double *__restrict__ p, int first, int step, int len,
                                double &M, double &sum)
{
    double mx = -INFINITY, sm = 0.0;
#pragma unroll 1
    for (int e = first; e < len; e += step) lse_step((double)k[e] + p[e], mx, sm);
    M = wave_max(mx);
    sum = wave_sum(mx > -INFINITY ? sm * exp(mx - M) : 0.0);
}

// Rows of C pieces of 1024 columns, the last piece not empty.
template <int C, int RG>
__global__ __launch_bounds__(DI_THREADS) void dense_rows_kernel(PassSide S, float *__restrict__ column_part,
                                                                unsigned long long *counters, int backward)
{
    __shared__ double sums[2][RG][DI_WAVES];
    __shared__ double wide[DI_WAVES][2];
    // what log v_j - base loses in single precision, each thread's own: kept here for the end, where a second trip to
    // memory for log v would cost 2 us
    __shared__ float lost_sh[C][DI_THREADS];
    const unsigned tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rows = (int)S.rows, cols = (int)S.rows_in;
    const int stride = gridDim.x * RG, step = backward ? -stride : stride;
    const unsigned last_piece = cols - DI_THREADS * (C - 1);   // 1 .. 1024 columns
    const bool in_last = tid < last_piece;
    // a lane past the end reads the last column and weighs it with zero
    const unsigned tid_last = in_last ? tid : last_piece - 1;
    unsigned long long empty = 0;
    bool missing = false, any_bad = false;

    auto load_values = [&](int r0, float (&k)[RG][C]) {
#pragma unroll
        for (int i = 0; i < RG; ++i) {   // rows past either end repeat the row there and count for nothing
            const int row = r0 + i < rows ? r0 + i : rows - 1;
            const float *__restrict__ kr = S.vals + (long long)(row > 0 ? row : 0) * cols;
#pragma unroll
            for (int c = 0; c < C; ++c) k[i][c] = (kr + DI_THREADS * c)[c == C - 1 ? tid_last : tid];
        }
    };
    // lane i < RG of every wavefront: what row i of the group needs
    auto load_record = [&](int r0, double &log_marg, double &log_u, float &marg) {
        int row = r0 + (lane < RG ? lane : RG - 1);
        row = row < rows ? row : rows - 1;
        const int *rec = S.meta + (long long)row * S.meta_stride;
        marg = __int_as_float(rec[2]);
        log_marg = __hiloint2double(rec[5], rec[4]);
        log_u = S.lin_out[row];
    };
    float ka[RG][C], kb[RG][C], pf[C], acc[C];
    const int first = blockIdx.x * RG, groups = first < rows ? (rows - first + stride - 1) / stride : 0;
    const int start = backward && groups ? first + (groups - 1) * stride : first;
    // One fp64 reference for the workgroup's shifts and for log v, their differences in single precision: a log v
    // itself, as what a column's difference loses is not seen by the rows.  `typical`: the shift of a row with mass.
    double base, typical;
    auto first_finite = [&](double x) {   // 0 if no lane has one
        const unsigned long long usable = __ballot(x > -INFINITY && x < INFINITY);
        const int from = usable ? __ffsll(usable) - 1 : 0;
        const double v = lane_value(x, from);
        return usable ? v : 0.0;
    };
    {
        double log_marg, log_u;
        float marg;
        load_record(first, log_marg, log_u, marg);
        typical = first_finite(log_marg - log_u);
        base = first_finite(S.perm_in[lane < cols ? lane : cols - 1]);
    }
    load_values(start, ka);
#pragma unroll
    for (int c = 0; c < C; ++c) {
        const double p = (S.perm_in + DI_THREADS * c)[c == C - 1 ? tid_last : tid];
        pf[c] = c == C - 1 && !in_last ? -INFINITY : (float)(p - base);
        acc[c] = 0.f;
        const double lost = p - base - (double)pf[c];
        lost_sh[c][tid] = fabs(lost) < 1.0 ? (float)lost : 0.f;
    }

    // Near the fixed point the factors of all rows with equal marginals round alike, iteration after iteration, and
    // so may the products and sums they go into: a common part would add up (u up, v down, 9e-9 per iteration at
    // 10 000 coinciding points a side).  Exactly, the rows' shares of the column sums add up to their masses,
    // t_i a_i / t_i; the workgroup keeps those masses and hands on by how much its column sums miss them.  For the
    // same reason the logarithms are double precision ones.
    double mass = 0.0;   // lane i < RG: of the rows it has seen
    auto group = [&](int r0, int buf, float (&k)[RG][C], float (&kn)[RG][C]) {
        double log_marg, log_u;
        float marg;
        load_record(r0, log_marg, log_u, marg);
        load_values(r0 + step, kn);
        // a row without mass only has to show that its sum is not empty: any shift does
        const double wanted = marg == 0.f ? typical : log_marg - log_u;
        // a shift that cannot be used: terms of zero
        const float off_l = wanted > -INFINITY && wanted < INFINITY ? (float)(wanted - base) : INFINITY;
        const double shift = base + (double)off_l;   // as the terms have it: its rounding is no error of the row
#pragma unroll
        for (int i = 0; i < RG; ++i) {
            const float off = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(off_l), i));
            float s = 0.f;
#pragma unroll
            for (int c = 0; c < C; ++c) {
                k[i][c] = __expf(k[i][c] + (pf[c] - off));
                s += k[i][c];
            }
            const double tot = wave_sum((double)s);
            if (lane == 0) sums[buf][i][wave] = tot;
        }
        lds_barrier();   // the buffer is written again two groups on, behind the next group's barrier
        double tot = 0.0;   // lane i < RG: row i's sum
#pragma unroll
        for (int w = 0; w < DI_WAVES; ++w) tot += sums[buf][lane < RG ? lane : RG - 1][w];
        const bool good = (tot > DI_ROW_MIN || (marg == 0.f && tot > 0.0)) && tot < DI_MAX && shift > -INFINITY &&
                          shift < INFINITY;
        // The same in every wavefront: the rows of this workgroup are written by it alone, behind the barrier.  Rows
        // past the end do not count: their stand-in, the last row, is another workgroup's to write meanwhile.
        any_bad = any_bad || __ballot(!good && lane < RG && r0 + lane < rows) != 0;
        // the column sums are taken times the number of columns: of order one
        float f_l = 0.f;
        if (lane < RG && r0 + lane < rows && good && marg != 0.f) {
            const double w = (double)marg * (double)cols;
            f_l = (float)(w * fast_rcp(tot));
            mass += w;
        }
#pragma unroll
        for (int i = 0; i < RG; ++i) {
            const float f = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(f_l), i));
#pragma unroll
            for (int c = 0; c < C; ++c) acc[c] = fmaf(k[i][c], f, acc[c]);
        }
        if (wave == 0 && lane < RG && r0 + lane < rows) {
            const int row = r0 + lane;
            const double lg = log_marg - (shift + short_log(tot));
            S.log_out[row] = good ? (float)lg : __builtin_nanf("");   // marked for the second look below
            if (good) {
                S.lin_out[row] = lg;
                S.perm_out[row] = lg;   // one bucket: its order is the points' own
            }
        }
    };
    if (groups)
        for (int r0 = start, left = groups;;) {
            group(r0, 0, ka, kb);
            if (--left == 0) break;
            r0 += step;
            group(r0, 1, kb, ka);
            if (--left == 0) break;
            r0 += step;
        }
    float *part = column_part + (long long)blockIdx.x * cols, *lost_out = column_part + (long long)gridDim.x * cols;
    double have = 0.0;   // what this thread's column sums hold of the mass
#pragma unroll
    for (int c = 0; c < C; ++c)
        if (c < C - 1 || in_last) {
            // what log v - base lost in single precision, the same in every workgroup, is a factor of the whole sum
            const float lost = lost_sh[c][tid];
            have += fma((double)acc[c], (double)lost, (double)acc[c]);
            (part + DI_THREADS * c)[tid] = acc[c];
            if (blockIdx.x == 0) (lost_out + DI_THREADS * c)[tid] = lost;
        }
    if (any_bad) {   // the marked rows' log-sum-exp with running maxima
        __syncthreads();
        for (int r0 = first; r0 < rows; r0 += stride)
            for (int row = r0; row < r0 + RG && row < rows; ++row) {
                if (S.log_out[row] == S.log_out[row]) continue;   // the same in every thread
                double M, sm;
                wave_lse(S.vals + (long long)row * cols, S.perm_in, (int)tid, DI_THREADS, cols, M, sm);
                if (lane == 0) {
                    wide[wave][0] = M;
                    wide[wave][1] = sm;
                }
                __syncthreads();   // and every thread has seen the mark
                if (tid == 0) {
                    M = -INFINITY;
                    for (int w = 0; w < DI_WAVES; ++w) M = fmax(M, wide[w][0]);
                    sm = 0.0;
                    for (int w = 0; w < DI_WAVES; ++w)
                        if (wide[w][0] > -INFINITY) sm += wide[w][1] * exp(wide[w][0] - M);
                    const int *rec = S.meta + (long long)row * S.meta_stride;
                    double lg;
                    if (sm > 0.0) {
                        lg = __hiloint2double(rec[5], rec[4]) - (M + log(sm));
                        // the row is missing from the column sums: without mass it would add nothing
                        if (__int_as_float(rec[2]) != 0.f) missing = true;
                    } else {  // no kernel entry reaches this point: it carries no mass
                        lg = -INFINITY;
                        ++empty;
                    }
                    S.log_out[row] = (float)lg;
                    S.lin_out[row] = lg;
                    S.perm_out[row] = lg;
                }
                __syncthreads();
            }
    }
    have = wave_sum(have);
    if (lane == 0) wide[wave][0] = have;
    __syncthreads();
    if (wave > 0) return;
    mass = wave_sum(mass);   // the same in every wavefront
    have = wave_sum(lane < DI_WAVES ? wide[lane < DI_WAVES ? lane : 0][0] : 0.0);
    if (lane == 0) {
        if (empty) atomicAdd(&counters[1], empty);
        // relative to the sums; a large one is no rounding (no rows, or a column's sum left the range, which
        // dense_columns_kernel sees for itself)
        const double off = mass / have - 1.0;
        lost_out[cols + blockIdx.x] = missing ? __builtin_nanf("") : fabs(off) < 1e-3 ? (float)off : 0.f;
    }
}

// v from the workgroups' column sums (column_part: a row of them per workgroup of dense_rows_kernel, then what the
// columns' log v lost in single precision, then per workgroup by how much its sums miss its rows' mass, relative to
// them, or NaN if it left a row out), 64 columns per workgroup.  A column whose sum left the range (a first
// iteration, a scaling that was infinite) takes its log-sum-exp from its row of the transpose.  A column without
// mass has no such sum either, but ends with a scaling of zero whatever it is: its row is read until one entry shows
// that it is not empty, mostly the first 64.
__global__ __launch_bounds__(DI_THREADS) void dense_columns_kernel(PassSide S, const float *__restrict__ column_part,
                                                                   int groups, unsigned long long *counters)
{
    __shared__ double sums[DI_WAVES][64];
    __shared__ double wide[64];
    __shared__ unsigned long long bad_sh, massless_sh;
    __shared__ int missing[DI_WAVES];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const long long j0 = (long long)blockIdx.x * 64;
    const long long j = j0 + lane < S.rows ? j0 + lane : S.rows - 1;
    // a workgroup left a row out of its sums: every column is taken from the transpose
    const float *__restrict__ lost = column_part + (long long)groups * S.rows, *__restrict__ off = lost + S.rows;
    double s = 0.0;
    bool left_out = false;
    for (int g0 = wave; g0 < groups; g0 += 16 * DI_WAVES) {   // every sixteenth group, sixteen of them in flight
        float part[16];
        const int of_lane = g0 + DI_WAVES * lane;
        const float off_l = lane < 16 && of_lane < groups ? off[of_lane] : 0.f;   // lane i: of the i-th
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int g = g0 + DI_WAVES * i;
            part[i] = column_part[(long long)(g < groups ? g : groups - 1) * S.rows + j];
        }
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const double p = g0 + DI_WAVES * i < groups ? (double)part[i] : 0.0;
            s += fma(p, (double)__int_as_float(__builtin_amdgcn_readlane(__float_as_int(off_l), i)), p);
        }
        left_out = left_out || __ballot(!(off_l == off_l)) != 0;
    }
    sums[wave][lane] = s;
    if (lane == 0) missing[wave] = left_out;   // a workgroup left a row out of its sums
    __syncthreads();
    double lse = 0.0, log_marg = 0.0;
    if (wave == 0) {
        s = 0.0;
#pragma unroll
        for (int w = 0; w < DI_WAVES; ++w) s += sums[w][lane];
        const int *rec = S.meta + j * S.meta_stride;
        log_marg = __hiloint2double(rec[5], rec[4]);
        const double prev = S.lin_out[j];
        const bool complete = __ballot(missing[lane < DI_WAVES ? lane : 0] != 0) == 0;
        const bool good = complete && s > DI_COLUMN_MIN && s < DI_MAX && prev > -INFINITY && prev < INFINITY;
        lse = log(s * (1.0 + (double)lost[j]) / (double)S.rows) - prev;
        const unsigned long long bad = __ballot(!good && j0 + lane < S.rows);
        const unsigned long long massless = __ballot(log_marg == -INFINITY);
        if (lane == 0) {
            bad_sh = bad;
            massless_sh = massless;
        }
    }
    __syncthreads();
    const unsigned long long bad = bad_sh;
    if (bad) {   // the same in every thread
        for (int i = wave; i < 64; i += DI_WAVES) {
            if (!(bad >> i & 1)) continue;
            if (massless_sh >> i & 1) {
                bool some = false;
                for (long long e0 = 0; e0 < S.rows_in && !some; e0 += 64) {
                    const long long e = e0 + lane < S.rows_in ? e0 + lane : S.rows_in - 1;
                    some = __ballot((double)S.vals[(j0 + i) * S.rows_in + e] + S.perm_in[e] > -INFINITY) != 0;
                }
                if (lane == 0) wide[i] = some ? 0.0 : -INFINITY;
                continue;
            }
            double M, sm;
            wave_lse(S.vals + (j0 + i) * S.rows_in, S.perm_in, lane, 64, (int)S.rows_in, M, sm);
            if (lane == 0) wide[i] = sm > 0.0 ? M + log(sm) : -INFINITY;
        }
        __syncthreads();
        if (wave == 0 && (bad >> lane & 1)) lse = wide[lane];
    }
    if (wave == 0) {
        unsigned long long empty = 0;
        if (j0 + lane < S.rows) {
            double lg;
            if (lse > -INFINITY) {
                lg = log_marg - lse;
            } else {  // no kernel entry reaches this point: it carries no mass
                lg = -INFINITY;
                ++empty;
            }
            S.log_out[j] = (float)lg;
            S.lin_out[j] = lg;
            S.perm_out[j] = lg;
        }
        empty = (unsigned long long)wave_sum((double)empty);
        if (lane == 0 && empty) atomicAdd(&counters[2], empty);
    }
}

static constexpr int dense_rows_of(int c) { return c <= 3 ? 8 : c >= 12 ? 1 : 24 / c; }

// Where the matrix is small the two launches and the trip through the column sums cost what the second read of it
// does (us per iteration, half-iterations by themselves against this: 2000 x 2000 15.1 / 12.4, 1500 x 2049
// 14.5 / 12.9, 3000 x 1024 14.8 / 13.3, 1000 x 3073 15.2 / 13.1, 46 000 x 70 102 / 72, 3500 x 3501 24.6 / 21.7, 4000 x 4000
// 29 / 22.8, 300 x 18 000 47 / 22, 10 000 x 10 000 159 / 80, 200 000 x 64 424 / 286); beyond 18 pieces a thread's
// registers are full.
int dense_iteration_groups(long long n, long long m, int cus)
{
    const bool worth = m <= DENSE_ITERATION_MAX_COLUMNS && n * m >= DENSE_ITERATION_MIN_PAIRS;
    return worth ? cus : 0;
}

hipError_t launch_dense_iteration(const PassSide &X, const PassSide &Y, Handle &h, hipStream_t s)
{
    const int c = (int)((h.m + DI_THREADS - 1) / DI_THREADS);
    const dim3 grid(h.column_groups), block(DI_THREADS);
#define LCN_DENSE_ROWS(C)                                                                                             \
    case C:                                                                                                          \
        hipLaunchKernelGGL((dense_rows_kernel<C, dense_rows_of(C)>), grid, block, 0, s, X, h.column_part, h.counters,   \
                           h.dense_backward);                                                                        \
        break
    switch (c) {
        LCN_DENSE_ROWS(1);
        LCN_DENSE_ROWS(2);
        LCN_DENSE_ROWS(3);
        LCN_DENSE_ROWS(4);
        LCN_DENSE_ROWS(5);
        LCN_DENSE_ROWS(6);
        LCN_DENSE_ROWS(7);
        LCN_DENSE_ROWS(8);
        LCN_DENSE_ROWS(9);
        LCN_DENSE_ROWS(10);
        LCN_DENSE_ROWS(11);
        LCN_DENSE_ROWS(12);
        LCN_DENSE_ROWS(13);
        LCN_DENSE_ROWS(14);
        LCN_DENSE_ROWS(15);
        LCN_DENSE_ROWS(16);
        LCN_DENSE_ROWS(17);
        LCN_DENSE_ROWS(18);
        default: return hipErrorInvalidValue;
    }
#undef LCN_DENSE_ROWS
    hipLaunchKernelGGL(dense_columns_kernel, dim3((unsigned)((h.m + 63) / 64)), block, 0, s, Y, h.column_part,
                       h.column_groups, h.counters);
    h.dense_backward ^= 1;
    return hipGetLastError();
}

}  // namespace lcn
