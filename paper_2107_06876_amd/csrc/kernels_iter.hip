// The half-iteration's host side, the sweeps of kernels held as logs (sparse, dense) and the reduction of the
// partial sums; the sweeps with factors are in sweep.h and kernels_sweep_long.hip.
#include <atomic>

#include "iter_common.h"
#include "log_walk.h"

namespace lcn {

// The half-iteration for kernels without signed parts (sparse K^sp, and the
// dense kernel as its one-bucket case), entirely in logs: the stored values
// are log K_ij = -C_ij / lambda, the vectors are log scalings, and a row's sum
// is a log-sum-exp (App. "Implementational details") with a running maximum per
// lane, so that scalings may drift arbitrarily far (a sparse kernel need not
// have support, App. "Limitations") without over- or underflow.
//
// G lanes work on a row (16, 32 or 64), a workgroup on 256 / G rows, and an update has a workgroup for
// every 256 / G rows there are: nothing is carried from row to row, so it is the chip that refills its compute units.
// The record is walked G U entries at a time, all loads of a trip requested together.  Flat (see pass_kernel), every entry's
// round is looked up: 34 vector instructions per 64 entries of three rounds.  Round by round that falls away, half of the
// instructions, the loads at fixed distances from the lane's first; but every round is a trip, or several, of its own.  Lanes past the
// round's end read on (the next values, the next places or what lies behind them in the workspace) and count as
// log K = -infinity.  log_walk.h says which is taken where.
// What bounds it: rows of some twenty entries, the launch and three trips to memory one after the other (record,
// values and scalings, stores); rows of some hundred entries, the trips and the values.
template <int RR, int G, int U, int MODE, bool BY_ROUNDS>
__global__ __launch_bounds__(256) void logpass_kernel(PassSide S, int R, double *partial, unsigned long long *counters,
                                                      int empty_slot)
{
    constexpr int RPB = 256 / G;
    __shared__ double qsh[4][2];
    __shared__ int empty_rows;
    const int sub = threadIdx.x % G;
    double q0 = 0.0, q1 = 0.0;
    if (MODE == PASS_UPDATE) {
        if (threadIdx.x == 0) empty_rows = 0;
        __syncthreads();
    }
    // (Once in an update and for the initial copies, and written so: of a loop the compiler takes the constants of exp and log in
    // double out, 36 registers of every lane for what hardly any row needs.)
    long long r0 = (long long)blockIdx.x * RPB;
    do {
        long long row = r0 + (G == 64 ? __builtin_amdgcn_readfirstlane(threadIdx.x / G) : threadIdx.x / G);
        const bool exists = row < S.rows;
        if (!exists) row = S.rows - 1;   // worked on again, not written
        double lg;
        if (MODE == PASS_INIT) {
            lg = (double)S.log_out[row];
        } else {
            // what takes an entry's number to its place in the gathered vector: place[r] in round r, or, where the record is
            // walked flat, place[0], and from the end of every round on place[r] more
            static_assert(!BY_ROUNDS || (G != 64 && RR <= EXACT_ROUNDS), "the ends of all rounds are in registers");
            long long base;
            float marg;
            double log_marg;
            int end[RR];
            unsigned place[RR];
            RecordWalk<ANY_ROUNDS> words{};   // of a wavefront's one row instead
            {
                const int *rec = S.meta + row * S.meta_stride;
                base = ((long long)rec[1] << 32) | (unsigned)rec[0];
                marg = __int_as_float(rec[2]);
                log_marg = __hiloint2double(rec[5], rec[4]);
                if (G == 64) load_walk<ANY_ROUNDS>(words, S, R, row);
                unsigned before = 0u;
#pragma unroll
                for (int r = 0; r < (G == 64 ? 0 : RR); ++r) {
                    const unsigned shift = (unsigned)rec[6 + 2 * r];
                    place[r] = BY_ROUNDS ? shift : shift - before;
                    before = shift;
                    const int e = rec[7 + 2 * r];
                    end[r] = RR <= EXACT_ROUNDS || r < R ? e : end[r > 0 ? r - 1 : 0];
                }
            }
            const double prev = S.lin_out[row];   // what the row's current scaling was computed from
            const float *__restrict__ vals = S.vals + base;
            const int total = G == 64 ? record_total<ANY_ROUNDS>(words, R) : end[RR - 1];
            // f(log kernel values, log scalings, entries that are left from this lane's first on) for pieces of G entries
            auto walk = [&](auto &&f) {
                if constexpr (BY_ROUNDS) {
                    static_assert(G * U <= VALUE_SLACK && 2 * G * U <= 2 * VALUE_SLACK, "read past the last record or place");
#pragma unroll
                    for (int r = 0; r < RR; ++r)
#pragma unroll 1
                        for (int e0 = r > 0 ? end[r > 0 ? r - 1 : 0] : 0; e0 < end[r]; e0 += G * U) {
                            const unsigned e = (unsigned)(e0 + sub);
                            const float *__restrict__ v = vals + e;
                            const double *__restrict__ q = S.perm_in + (e + place[r]);
                            float k[U];
                            double p[U];
#pragma unroll
                            for (int u = 0; u < U; ++u) {
                                k[u] = v[G * u];
                                p[u] = q[G * u];
                            }
                            f(k, p, end[r] - e0 - sub);
                        }
                } else {
                    RecordCursor<ANY_ROUNDS> cursor(words, R);
                    for (int e0 = 0; e0 < total; e0 += G * U) {
                        float k[U];
                        double p[U];
#pragma unroll
                        for (int u = 0; u < U; ++u) {
                            int e = e0 + G * u + sub;
                            unsigned at;
                            if constexpr (G == 64) at = cursor.place(e0 + G * u, e, 0u);
                            e = e < total ? e : total - 1;   // past the end: the last entry again, not counted
                            if constexpr (G != 64) {
                                at = (unsigned)e + place[0];
#pragma unroll
                                for (int r = 1; r < RR; ++r) at += e >= end[r - 1] ? place[r] : 0u;
                            }
                            k[u] = vals[(unsigned)e];
                            p[u] = S.perm_in[at];
                        }
                        f(k, p, total - e0 - sub);
                    }
                }
            };
            auto sum_lanes = [&](double v) { return G == 64 ? wave_sum(v) : G == 32 ? half_sum(v) : row_sum(v); };
            // The row's log-sum-exp.  First with the row's previous value as the shift (near the answer, so the
            // terms are of order one): one subtraction, one single-precision exp and one addition in double per entry (a
            // lane has up to four times the entries it would have if a wavefront shared the row: added in single precision,
            // 510 entries per row, 200 iterations, the scalings' logs were off by 6.9e-6, root mean square).  If that
            // shift is unusable (no previous value, or the sum leaves single precision's range) the row is walked again
            // with a running maximum per lane, which cannot over- or underflow.
            const double shift = log_marg - prev;
            double lse = 0.0;
            bool done = false;
            if (shift > -INFINITY && shift < INFINITY) {   // the same in every lane of the row
                double acc = 0.0;
                walk([&](const auto &k, const auto &p, int left) {
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const float x = k[u] + (float)(p[u] - shift);
                        acc += (double)__expf(G * u < left ? x : -INFINITY);
                    }
                });
                const double tot = sum_lanes(acc);
                if (tot > 1e-30 && tot < 1e30) {
                    lse = shift + fast_log(tot);
                    done = true;
                }
            }
            if (!done) {
                double mx = -INFINITY, sm = 0.0;
                if constexpr (BY_ROUNDS) {
#pragma unroll 1
                    for (int e = sub; e < total; e += G) {
                        unsigned at = (unsigned)e + place[0];
#pragma unroll
                        for (int r = 1; r < RR; ++r) at = e >= end[r - 1] ? (unsigned)e + place[r] : at;
                        lse_step((double)vals[(unsigned)e] + S.perm_in[at], mx, sm);
                    }
                } else {
                    walk([&](const auto &k, const auto &p, int left) {
#pragma unroll
                        for (int u = 0; u < U; ++u) lse_step(G * u < left ? (double)k[u] + p[u] : -INFINITY, mx, sm);
                    });
                }
                const double M = G == 64 ? wave_max(mx) : G == 32 ? half_max(mx) : row_max(mx);
                const double part = mx > -INFINITY ? sm * exp(mx - M) : 0.0;
                const double ssum = sum_lanes(part);
                lse = ssum > 0.0 ? M + log(ssum) : -INFINITY;
            }
            if (MODE == PASS_UPDATE) {
                if (lse > -INFINITY) {
                    lg = log_marg - lse;
                } else {  // no kernel entry reaches this point: it carries no mass
                    lg = -INFINITY;
                    if (exists && sub == 0) atomicAdd(&empty_rows, 1);
                }
                if (exists && sub == 0) S.log_out[row] = (float)lg;
            } else {  // PASS_QUERY
                lg = prev;
                const double ri = (lg > -INFINITY && lse > -INFINITY) ? exp(lg + lse) : 0.0;
                if (exists && sub == 0) {
                    if (S.marg_out) S.marg_out[row] = (float)ri;
                    if (ri != 0.0) q0 += ri * lg;
                    q1 += fabs(ri - (double)marg);
                }
            }
        }
        if (MODE != PASS_QUERY && exists) {
            if (sub == 0) S.lin_out[row] = lg;
            if (sub < R) S.perm_out[(long long)sub * S.rows + S.meta[row * S.meta_stride + 6 + 2 * R + sub]] = lg;
        }
        r0 += (long long)gridDim.x * RPB;
    } while (MODE == PASS_QUERY && r0 < S.rows);
    if (MODE == PASS_QUERY) {
        q0 = wave_sum(q0);
        q1 = wave_sum(q1);
        if ((threadIdx.x & 63) == 0) {
            qsh[threadIdx.x >> 6][0] = q0;
            qsh[threadIdx.x >> 6][1] = q1;
        }
        __syncthreads();
        if (threadIdx.x < 3) {
            double s = threadIdx.x == 2 ? -INFINITY : 0.0;
            if (threadIdx.x < 2)
                for (int w = 0; w < 4; ++w) s += qsh[w][threadIdx.x];
            partial[(long long)blockIdx.x * 3 + threadIdx.x] = s;
        }
    }
    if (MODE == PASS_UPDATE) {
        __syncthreads();
        if (threadIdx.x == 0 && empty_rows) atomicAdd(&counters[empty_slot], (unsigned long long)empty_rows);
    }
}

// The dense kernel (one bucket, one round): every row multiplies the same vector, so a workgroup
// takes DENSE_ROWS consecutive rows and reads each piece of the vector once for all of them
// (one row per wavefront reads it once per row: twice the bytes of the kernel matrix itself,
// from cache).  Its DENSE_WAVES wavefronts share out the columns in pieces of 128 and merge their
// running (maximum, scaled sum) pairs through LDS.  Otherwise as logpass_kernel; PASS_INIT stays
// with logpass_kernel.
constexpr int DENSE_ROWS = 8;
constexpr int DENSE_WAVES = 4;

template <int MODE>
__global__ __launch_bounds__(64 * DENSE_WAVES) void logpass_dense_kernel(PassSide S, double *partial,
                                                                         unsigned long long *counters, int empty_slot)
{
    __shared__ double msh[DENSE_WAVES][DENSE_ROWS][2];
    __shared__ int flag;   // some row of the group needs the second pass
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    double q0 = 0.0, q1 = 0.0;
    unsigned long long empty = 0;
    for (long long r0 = (long long)blockIdx.x * DENSE_ROWS; r0 < S.rows; r0 += (long long)gridDim.x * DENSE_ROWS) {
        RowMeta<1> mt[DENSE_ROWS];
#pragma unroll
        for (int i = 0; i < DENSE_ROWS; ++i)   // rows past the end repeat the last row and are dropped below
            load_meta<1, MODE>(mt[i], S, 1, r0 + i < S.rows ? r0 + i : S.rows - 1, lane);
        const int len = mt[0].walk.end[0];
        const double *__restrict__ vp = S.perm_in + mt[0].walk.shift[0];
        // two wavefront-wide pieces per trip; the next trip's loads are requested before this trip's
        // values are used
        auto fetch = [&](int e0, double (&p)[2], float (&k)[DENSE_ROWS][2]) {
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const int e = e0 + 64 * q;
                const bool in = e < len;
                p[q] = in ? vp[e] : -INFINITY;
#pragma unroll
                for (int i = 0; i < DENSE_ROWS; ++i) k[i][q] = in ? S.vals[mt[i].base + e] : 0.f;
            }
        };
        // f(row of the group, log kernel value, log scaling, piece) for this wavefront's share of the columns
        auto walk = [&](auto &&f) {
            double pv[2], pvn[2];
            float kv[DENSE_ROWS][2], kvn[DENSE_ROWS][2];
            fetch(128 * wave + lane, pv, kv);
            for (int e0 = 128 * wave + lane; e0 < len; e0 += 128 * DENSE_WAVES) {
                fetch(e0 + 128 * DENSE_WAVES, pvn, kvn);   // beyond the row: nothing is read
                f(kv, pv);
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    pv[q] = pvn[q];
#pragma unroll
                    for (int i = 0; i < DENSE_ROWS; ++i) kv[i][q] = kvn[i][q];
                }
            }
        };
        // First pass: every row's previous log-sum-exp as its shift (see logpass_kernel), sums in single
        // precision; shifts as one common fp64 base plus a small per-row offset.
        double shift[DENSE_ROWS];
        bool usable = true;
#pragma unroll
        for (int i = 0; i < DENSE_ROWS; ++i) {
            const long long row = r0 + i < S.rows ? r0 + i : S.rows - 1;
            shift[i] = mt[i].log_marg - (MODE == PASS_QUERY ? mt[i].lin : S.lin_out[row]);
            usable = usable && shift[i] > -INFINITY && shift[i] < INFINITY;
        }
        __syncthreads();   // the previous group's merge has read msh and flag
        if (usable) {   // the same in every thread
            float off[DENSE_ROWS], accf[DENSE_ROWS];
#pragma unroll
            for (int i = 0; i < DENSE_ROWS; ++i) {
                off[i] = (float)(shift[i] - shift[0]);
                accf[i] = 0.f;
            }
            walk([&](const float (&kv)[DENSE_ROWS][2], const double (&pv)[2]) {
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const float pf = (float)(pv[q] - shift[0]);
#pragma unroll
                    for (int i = 0; i < DENSE_ROWS; ++i) accf[i] += __expf(kv[i][q] + (pf - off[i]));
                }
            });
#pragma unroll
            for (int i = 0; i < DENSE_ROWS; ++i) {
                const double tot = wave_sum((double)accf[i]);
                if (lane == 0) msh[wave][i][0] = tot;
            }
        }
        if (threadIdx.x == 0) flag = usable ? 0 : 1;
        __syncthreads();
        double lse = 0.0;   // wavefront 0, lane i: row r0 + i
        if (usable && wave == 0 && lane < DENSE_ROWS) {
            double tot = 0.0;
#pragma unroll
            for (int w = 0; w < DENSE_WAVES; ++w) tot += msh[w][lane][0];
            double sh_l = shift[0];
#pragma unroll
            for (int i = 1; i < DENSE_ROWS; ++i) sh_l = lane == i ? shift[i] : sh_l;
            if (tot > 1e-30 && tot < 1e30)
                lse = sh_l + fast_log(tot);
            else if (r0 + lane < S.rows)
                flag = 1;   // benign race: every writer stores 1
        }
        __syncthreads();
        if (flag) {   // the same in every thread: some sum left single precision's range, walk again with running maxima
            double mx[DENSE_ROWS], sm[DENSE_ROWS];
#pragma unroll
            for (int i = 0; i < DENSE_ROWS; ++i) {
                mx[i] = -INFINITY;
                sm[i] = 0.0;
            }
            walk([&](const float (&kv)[DENSE_ROWS][2], const double (&pv)[2]) {
#pragma unroll
                for (int q = 0; q < 2; ++q)
#pragma unroll
                    for (int i = 0; i < DENSE_ROWS; ++i) lse_step((double)kv[i][q] + pv[q], mx[i], sm[i]);
            });
#pragma unroll
            for (int i = 0; i < DENSE_ROWS; ++i) {
                const double M = wave_max(mx[i]);
                const double part = mx[i] > -INFINITY ? sm[i] * exp(mx[i] - M) : 0.0;
                const double ssum = wave_sum(part);
                if (lane == 0) {
                    msh[wave][i][0] = M;
                    msh[wave][i][1] = ssum;
                }
            }
            __syncthreads();
            if (wave == 0 && lane < DENSE_ROWS) {
                double M = -INFINITY;
#pragma unroll
                for (int w = 0; w < DENSE_WAVES; ++w) M = fmax(M, msh[w][lane][0]);
                double ssum = 0.0;
#pragma unroll
                for (int w = 0; w < DENSE_WAVES; ++w)
                    if (msh[w][lane][0] > -INFINITY) ssum += msh[w][lane][1] * exp(msh[w][lane][0] - M);
                lse = ssum > 0.0 ? M + log(ssum) : -INFINITY;
            }
        }
        // wavefront 0, lane i finishes row r0 + i
        if (wave == 0 && lane < DENSE_ROWS && r0 + lane < S.rows) {
            const long long row = r0 + lane;
            // this lane's row record (the registers hold it per row index, which is a lane here)
            const int *rec = S.meta + row * S.meta_stride;
            if (MODE == PASS_UPDATE) {
                const double log_marg = __hiloint2double(rec[5], rec[4]);
                double lg;
                if (lse > -INFINITY) {
                    lg = log_marg - lse;
                } else {  // no kernel entry reaches this point: it carries no mass
                    lg = -INFINITY;
                    ++empty;
                }
                S.log_out[row] = (float)lg;
                S.lin_out[row] = lg;
                S.perm_out[rec[6 + 2 * 1]] = lg;   // one round: the row's position in the bucket order
            } else {  // PASS_QUERY
                const double lg = S.lin_out[row];
                const double ri = (lg > -INFINITY && lse > -INFINITY) ? exp(lg + lse) : 0.0;
                if (S.marg_out) S.marg_out[row] = (float)ri;
                if (ri != 0.0) q0 += ri * lg;
                q1 += fabs(ri - (double)__int_as_float(rec[2]));
            }
        }
    }
    if (MODE == PASS_QUERY) {
        // only wavefront 0 holds terms, one row per lane
        q0 = wave_sum(q0);
        q1 = wave_sum(q1);
        if (threadIdx.x == 0) {
            partial[(long long)blockIdx.x * 3 + 0] = q0;
            partial[(long long)blockIdx.x * 3 + 1] = q1;
            partial[(long long)blockIdx.x * 3 + 2] = -INFINITY;
        }
    }
    empty = (unsigned long long)wave_sum((double)empty);
    if (threadIdx.x == 0 && empty) atomicAdd(&counters[empty_slot], empty);
}

// Adds the per-workgroup partial sums of a sweep in a fixed order (so the
// result does not depend on timing), 16 columns per workgroup.
// Entry lp + 2 is a maximum (the largest log scaling of the sweep), which
// becomes this side's exponent for the next sweep; entry lp of the output
// accumulator records the exponent that this sweep's vector was stored with.
__global__ __launch_bounds__(1024) void reduce_partials_kernel(const double *__restrict__ partial, int groups,
                                                               int stride, int lp, double *acc_out,
                                                               double *query_out, double *shift_self, int mode)
{
    __shared__ double red[64 * REDUCE_COLUMNS];
    const double s = reduce_columns(partial, groups, stride, blockIdx.x, lp + 2, red);
    const int k = REDUCE_COLUMNS * blockIdx.x + threadIdx.x;
    if (threadIdx.x < REDUCE_COLUMNS && k < stride) {
        if (k < lp) {
            if (mode != PASS_QUERY) acc_out[k] = s;
        } else if (k < lp + 2) {
            if (mode == PASS_QUERY) query_out[k - lp] = s;
        } else if (mode != PASS_QUERY) {
            acc_out[lp] = *shift_self;                              // exponent used by this sweep
            *shift_self = (s > -INFINITY && s < INFINITY) ? s : 0.0;  // exponent for the next one
        }
    }
}

// largest finite entry of a float vector (0 if there is none); one workgroup
__global__ __launch_bounds__(1024) void max_log_kernel(const float *__restrict__ x, long long n, double *out)
{
    __shared__ float sh[1024];
    float m = -INFINITY;
    for (long long i = threadIdx.x; i < n; i += 1024) {
        const float v = x[i];
        if (v > m && v < INFINITY) m = v;
    }
    sh[threadIdx.x] = m;
    __syncthreads();
    for (int o = 512; o > 0; o >>= 1) {
        if (threadIdx.x < o) sh[threadIdx.x] = fmaxf(sh[threadIdx.x], sh[threadIdx.x + o]);
        __syncthreads();
    }
    if (threadIdx.x == 0) *out = sh[0] > -INFINITY ? (double)sh[0] : 0.0;
}

// Workgroups of a sweep: as many as are resident at once (compute units x
// workgroups per compute unit that the kernel's register use allows), so that
// every row slot is dealt out once and the partial sums stay few.
int device_compute_units()
{
    static std::atomic<int> known[64];   // per device, looked up once (the query takes tens of microseconds)
    int dev = 0, cus = 256;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) {
        (void)hipGetLastError();
        return cus;
    }
    const int have = known[dev].load(std::memory_order_relaxed);
    if (have > 0) return have;
    int got = 0;
    if (hipDeviceGetAttribute(&got, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && got > 0) {
        cus = got;
        known[dev].store(cus, std::memory_order_relaxed);
    }
    (void)hipGetLastError();
    return cus;
}

// In logs these are the workgroups of a query (an update leaves no partial sums and has as many as it likes).  A sparse
// kernel's have four wavefronts, so it takes 2048 of them to fill the chip.
int pass_grid(const Handle &h)
{
    const long long rows = h.n > h.m ? h.n : h.m;
    const bool sparse = h.mode == LCN_MODE_SPARSE;
    const int each = sparse ? 4 : PASS_WAVES;
    const long long g = (rows + each - 1) / each;
    long long cap = h.grid_cap;
    if (cap <= 0) cap = sparse ? MOST_GROUPS : h.log_domain ? 512 : device_compute_units();
    return (int)(g < cap ? g : cap);
}

// Rows a wavefront takes at a time in a sweep with a sparse part: as many as give every wavefront of the chip one
// group (up to five), else three or five, whichever comes to fewer rows per wavefront.  1024 rows: one 5.5 us, two
// 5.8, three 6.1; 10 000 rows of 128 entries: two 13.6, three 11.6, five 13.6; 20 000 rows of 256: two 15.1, three
// 13.8, five 13.3 (eight spill).
int rows_at_a_time(const Handle &h, long long rows)
{
    if (h.lp > 256) return 1;
    const long long waves = (long long)PASS_WAVES * (h.cus > 0 ? h.cus : 256), each = (rows + waves - 1) / waves;
    if (each <= 3) return (int)each;
    if (each <= 5) return 5;
    const long long three = (rows + 3 * waves - 1) / (3 * waves) * 3, five = (rows + 5 * waves - 1) / (5 * waves) * 5;
    return three < five ? 3 : 5;
}

// workgroups of a sweep over `rows` rows (= partial sums it leaves)
static int sweep_groups(const Handle &h, long long rows)
{
    if (!h.log_domain && h.R == 0) return nystrom_sweep_groups(h, rows);
    const long long per = (long long)PASS_WAVES * rows_at_a_time(h, rows), g = (rows + per - 1) / per;
    return (int)(g < h.grid ? g : h.grid);
}

// side 0: rows of X (updates u, consumes y = W v, produces z = U^T u); side 1: rows of Y.
// acc_in / acc_out index the accumulator buffers (-1: none).
static PassSide make_side(const Handle &h, int side, int acc_in, int acc_out, float *marg_out)
{
    PassSide S;
    if (side == 0) {
        S.rows = h.n;
        S.F = h.U;
        S.vals = h.vals_x;
        S.meta = h.sort.meta_x;
        S.log_out = h.log_u;
        S.lin_out = h.lin_u;
        S.perm_out = h.perm_u;
        S.perm_in = h.perm_v;
        S.rows_in = h.m;
    } else {
        S.rows = h.m;
        S.F = h.Wt;
        S.vals = h.vals_y;
        S.meta = h.sort.meta_y;
        S.log_out = h.log_v;
        S.lin_out = h.lin_v;
        S.perm_out = h.perm_v;
        S.perm_in = h.perm_u;
        S.rows_in = h.n;
    }
    S.acc_in = acc_in >= 0 ? h.acc[acc_in] : nullptr;
    S.acc_out = acc_out >= 0 ? h.acc[acc_out] : nullptr;
    S.marg_out = marg_out;
    S.meta_stride = h.sort.meta_stride;
    S.shift_self = h.shift + 2 * side + h.shift_slot[side];
    return S;
}

template <int RR, int G, int U, bool BY_ROUNDS>
static int launch_log_update(const PassSide &S, const Handle &h, int empty_slot, hipStream_t s)
{
    const int grid = (int)((S.rows + 256 / G - 1) / (256 / G));
    hipLaunchKernelGGL((logpass_kernel<RR, G, U, PASS_UPDATE, BY_ROUNDS>), dim3(grid), dim3(256), 0, s, S, h.R, h.partial, h.counters,
                       empty_slot);
    return grid;
}

template <int RR, int G, int U, bool BY_ROUNDS>
static int launch_log_query(const PassSide &S, const Handle &h, int empty_slot, hipStream_t s)
{
    // A query leaves 3 partial sums per workgroup and there is room for h.grid of them.  Few entries are read faster than
    // many partial sums are added up (a query of both sides, 512 workgroups / as many as there is room for: 10 000 rows
    // of 167 values 38 / 43 us, 20 000 of 200 52 / 55, 20 000 of 250 72 / 65, 40 000 of 1200 212 / 178, with a wavefront per
    // row 30 000 of 2000 312 / 216).
    const long long all = (S.rows + 256 / G - 1) / (256 / G);
    const long long most = h.nnz_stored <= (1ll << 22) && h.grid > 512 ? 512 : h.grid;
    const int grid = (int)(all > most ? most : all);
    constexpr int LONG_U = G == 64 ? 8 : U;   // long rows, a wavefront each (40 000 of 1600 values 233 -> 197 us; of 140 82 -> 93)
    if (LONG_U != U && h.nnz_stored > 500 * S.rows)
        hipLaunchKernelGGL((logpass_kernel<RR, G, LONG_U, PASS_QUERY, BY_ROUNDS>), dim3(grid), dim3(256), 0, s, S, h.R, h.partial,
                           h.counters, empty_slot);
    else
        hipLaunchKernelGGL((logpass_kernel<RR, G, U, PASS_QUERY, BY_ROUNDS>), dim3(grid), dim3(256), 0, s, S, h.R, h.partial,
                           h.counters, empty_slot);
    return grid;
}

// RR rounds, the walk as log_walk() gives it for them; only what it gives is compiled.  Returns the workgroups launched.
template <int RR>
static int launch_log_walk(const PassSide &S, const Handle &h, LogWalk walk, bool query, int empty_slot, hipStream_t s)
{
#define LCN_LOG_WALK(G, U, BY_ROUNDS)                                             \
    (query ? launch_log_query<RR, G, U, BY_ROUNDS>(S, h, empty_slot, s) : launch_log_update<RR, G, U, BY_ROUNDS>(S, h, empty_slot, s))
    if constexpr (RR == ANY_ROUNDS) {
        if (walk == FLAT_16x2) return LCN_LOG_WALK(16, 2, false);
        if (walk == FLAT_64x4) return LCN_LOG_WALK(64, 4, false);
        return LCN_LOG_WALK(32, 4, false);
    } else if constexpr (RR == 1) {
        if (walk == ROUNDS_16x2) return LCN_LOG_WALK(16, 2, true);
        if (walk == ROUNDS_16x4) return LCN_LOG_WALK(16, 4, true);
        if (walk == ROUNDS_32x2) return LCN_LOG_WALK(32, 2, true);
        return LCN_LOG_WALK(32, 4, true);
    } else {
        if (walk == FLAT_16x2) return LCN_LOG_WALK(16, 2, false);
        if (walk == ROUNDS_32x4) return LCN_LOG_WALK(32, 4, true);
        if (walk == ROUNDS_32x2 && !query) return launch_log_update<RR, 32, 2, true>(S, h, empty_slot, s);
        if (walk == ROUNDS_16x4 && query) return launch_log_query<RR, 16, 4, true>(S, h, empty_slot, s);
        return LCN_LOG_WALK(32, 4, false);
    }
#undef LCN_LOG_WALK
}

static int launch_logpass_rows(const PassSide &S, const Handle &h, int mode, int empty_slot, hipStream_t s)
{
    if (mode == PASS_INIT) {
        const int grid = (int)((S.rows + 15) / 16);
        hipLaunchKernelGGL((logpass_kernel<1, 16, 1, PASS_INIT, false>), dim3(grid), dim3(256), 0, s, S, h.R, h.partial, h.counters,
                           empty_slot);
        return grid;
    }
    const bool query = mode == PASS_QUERY;
    const LogWalk walk = log_walk(h.R, S.rows, h.nnz_stored, query);
    if (walk == FLAT_64x4) return launch_log_walk<ANY_ROUNDS>(S, h, walk, query, empty_slot, s);
    switch (h.R) {
        case 1: return launch_log_walk<1>(S, h, walk, query, empty_slot, s);
        case 2: return launch_log_walk<2>(S, h, walk, query, empty_slot, s);
        case 3: return launch_log_walk<3>(S, h, walk, query, empty_slot, s);
        case 4: return launch_log_walk<4>(S, h, walk, query, empty_slot, s);
        default: return launch_log_walk<ANY_ROUNDS>(S, h, walk, query, empty_slot, s);
    }
}

static hipError_t launch_logpass(const PassSide &S, const Handle &h, int side, int mode, hipStream_t s)
{
    const int empty_slot = 1 + side;
    if (h.mode == LCN_MODE_DENSE && mode != PASS_INIT) {
        const long long gd = (S.rows + DENSE_ROWS - 1) / DENSE_ROWS;
        // a query leaves 3 partial sums per workgroup and there is room for h.grid of them; an update
        // leaves none and may fill every compute unit with eight of these small workgroups
        const long long cap = mode == PASS_QUERY ? (long long)h.grid : 8ll * (h.cus > 0 ? h.cus : 256);
        const int dgrid = (int)(gd < cap ? gd : cap);
        if (mode == PASS_UPDATE)
            hipLaunchKernelGGL(logpass_dense_kernel<PASS_UPDATE>, dim3(dgrid), dim3(64 * DENSE_WAVES), 0, s, S, h.partial,
                               h.counters, empty_slot);
        else
            hipLaunchKernelGGL(logpass_dense_kernel<PASS_QUERY>, dim3(dgrid), dim3(64 * DENSE_WAVES), 0, s, S, h.partial,
                               h.counters, empty_slot);
        if (mode == PASS_QUERY)
            hipLaunchKernelGGL(reduce_partials_kernel, dim3(1), dim3(1024), 0, s, h.partial, dgrid, 3, 0, S.acc_out,
                               h.query_out + 2 * side, S.shift_self, mode);
        return hipGetLastError();
    }
    const int grid = launch_logpass_rows(S, h, mode, empty_slot, s);
    if (mode == PASS_QUERY)
        hipLaunchKernelGGL(reduce_partials_kernel, dim3(1), dim3(1024), 0, s, h.partial, grid, 3, 0, S.acc_out,
                           h.query_out + 2 * side, S.shift_self, mode);
    return hipGetLastError();
}

static hipError_t dispatch_pass(const PassSide &S, const Handle &h, int side, int mode, const FuseArgs *fuse,
                                bool fused_in, bool reduce_after, double *partial, hipStream_t s,
                                unsigned long long *cnt = nullptr)
{
    if (!cnt) cnt = h.counters;
    hipError_t e = hipErrorInvalidValue;
    if (h.R == 0) {
        e = launch_nystrom_pass(S, h, mode, fuse, fused_in, partial, cnt, s);
    } else {
        const FuseArgs F = fuse ? *fuse : FuseArgs{};
        const int groups = sweep_groups(h, S.rows);
        if (h.lp <= 128)
            e = launch_short_sweep(S, h, mode, F, fused_in, groups, partial, cnt, s);
        else if (h.lp <= 256)
            e = launch_mid_sweep(S, h, mode, F, fused_in, groups, partial, cnt, s);
        else
            e = launch_long_sweep(S, h, mode, F, fused_in, groups, partial, cnt, s);
    }
    if (e != hipSuccess || !reduce_after) return e;
    const int stride = h.lp + 3;
    hipLaunchKernelGGL(reduce_partials_kernel, dim3((stride + REDUCE_COLUMNS - 1) / REDUCE_COLUMNS), dim3(1024), 0, s, partial,
                       sweep_groups(h, S.rows), stride, h.lp, S.acc_out, h.query_out + 2 * side, S.shift_self, mode);
    return hipGetLastError();
}

hipError_t launch_pass(const Handle &h, int side, int mode, int acc_in, int acc_out, float *marg_out, hipStream_t s)
{
    const PassSide S = make_side(h, side, acc_in, acc_out, marg_out);
    if (h.log_domain) return launch_logpass(S, h, side, mode, s);
    return dispatch_pass(S, h, side, mode, nullptr, false, true, h.partial, s);
}

hipError_t launch_init_pass(const Handle &h, int side, int acc_out, bool zero_logs, hipStream_t s)
{
    const PassSide S = make_side(h, side, -1, acc_out, nullptr);
    if (!h.log_domain && !zero_logs)   // the exponent to take out
        hipLaunchKernelGGL(max_log_kernel, dim3(1), dim3(1024), 0, s, S.log_out, S.rows, S.shift_self);
    return launch_pass(h, side, PASS_INIT, -1, acc_out, nullptr, s);
}

// `iters` iterations = 2 iters update sweeps (rows of X, then rows of Y).  With
// fused reduction every sweep but the first adds up its predecessor's partial
// sums itself (two partial buffers alternate) and one reduction launch at the end
// completes the state; otherwise every sweep is followed by its reduction launch.
//
// A state that has not been iterated yet (after the build or after new scalings
// were set) has exponents that say nothing about the vectors the first sweeps
// produce: from u = v = 1 the first u is of the order of 1 / (K 1), possibly
// e^(+-hundreds).  For such a state each side's first sweep is run twice: once
// only to learn the largest log of its result (everything else it writes is
// overwritten, its fault counts go to slots nobody reads), then for real with
// that exponent.  From then on a vector's exponent is its largest log one
// iteration earlier, and logs move little per iteration.
hipError_t launch_update_sweeps(Handle &h, int iters, hipStream_t s)
{
    const bool fused = h.fused_reduce && !h.log_domain;
    auto direct_into = [&](int side) {   // how the sweep over `side` takes the totals of the other side's
        return h.lp == 64 && sweep_groups(h, side == 0 ? h.m : h.n) <= DIRECT_GROUPS;
    };
    int first = 0;
    if (h.fresh && h.double_first && !h.log_domain && iters > 0) {
        unsigned long long *discard = h.counters + 8;
        const PassSide SX = make_side(h, 0, 0, 1, nullptr), SY = make_side(h, 1, 1, 0, nullptr);
        hipError_t e = dispatch_pass(SX, h, 0, PASS_UPDATE, nullptr, false, true, h.partial, s, discard);
        if (e == hipSuccess) e = dispatch_pass(SX, h, 0, PASS_UPDATE, nullptr, false, true, h.partial, s);
        if (e == hipSuccess) e = dispatch_pass(SY, h, 1, PASS_UPDATE, nullptr, false, true, h.partial, s, discard);
        if (e != hipSuccess) return e;
        first = 1;   // the loop below starts with the sweep over Y, now with its exponent known
    }
    h.last_launches = 2 * iters + (first ? 2 : 0);   // half-iterations of this run, the repeated ones included
    const bool fresh = h.fresh != 0;
    if (iters > 0) h.fresh = 0;
    if (bucket_run_taken(h)) return launch_bucket_run(make_side(h, 0, -1, -1, nullptr), make_side(h, 1, -1, -1, nullptr), h, iters, s);
    for (int t = first; t < 2 * iters; ++t) {
        const int side = t & 1;
        const PassSide S = make_side(h, side, side == 0 ? 0 : 1, side == 0 ? 1 : 0, nullptr);
        hipError_t e;
        if (h.column_part && side == 0 && !(fresh && t == 0)) {
            // dense: both halves of the iteration from one read of the kernel matrix.  Not for scalings that have
            // not been iterated: their shifts are far off and every row and column would be walked again.
            e = launch_dense_iteration(S, make_side(h, 1, 1, 0, nullptr), h, s);
            ++t;
        } else if (h.log_domain) {
            e = launch_logpass(S, h, side, PASS_UPDATE, s);
        } else if (!fused) {
            e = dispatch_pass(S, h, side, PASS_UPDATE, nullptr, false, true, h.partial, s);
        } else {
            double *mine = (t & 1) ? h.partial2 : h.partial;
            const bool last = t == 2 * iters - 1;
            if (t == first) {
                // not fused itself, but its successor reduces into this sweep's output accumulator
                FuseArgs F{};
                F.mark_pending = last || direct_into(1 - side) ? nullptr : h.acc[side == 0 ? 1 : 0];
                e = dispatch_pass(S, h, side, PASS_UPDATE, &F, false, last, mine, s);
            } else {
                const long long rows_prev = side == 0 ? h.m : h.n;
                FuseArgs F;
                F.prev_partial = (t & 1) ? h.partial : h.partial2;
                F.prev_groups = sweep_groups(h, rows_prev);
                F.direct = direct_into(side);
                F.acc = h.acc[side == 0 ? 0 : 1];
                F.shift_other = h.shift + 2 * (1 - side) + h.shift_slot[1 - side];
                F.shift_self = S.shift_self;
                h.shift_slot[1 - side] ^= 1;
                F.shift_next = h.shift + 2 * (1 - side) + h.shift_slot[1 - side];
                F.mark_pending = last || direct_into(1 - side) ? nullptr : h.acc[side == 0 ? 1 : 0];
                F.timeouts = h.counters + 5;
                F.wait_ticks = h.wait_ticks;
                e = dispatch_pass(S, h, side, PASS_UPDATE, &F, true, last, mine, s);
            }
        }
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace lcn
