// Device helpers of the half-iteration kernels: cross-lane sums, the short log and
// reciprocal used by the scaling update, the factor-row register layout and the
// in-kernel completion of the previous sweep's reduction.
#pragma once

#include "lcn_internal.h"

namespace lcn {

constexpr int PASS_THREADS = 1024;
constexpr int PASS_WAVES = PASS_THREADS / 64;
constexpr int MAXR = 8;
// what the single-precision bucket-ordered copies of a scaling vector are stored times, and its inverse
constexpr double PERM_SCALE = 18446744073709551616.0;          // 2^64
constexpr double PERM_UNSCALE = 1.0 / 18446744073709551616.0;  // 2^-64

__device__ inline double lane_value(double v, int src_lane)   // src_lane: the same in every lane
{
    const int lo = __builtin_amdgcn_readlane(__double2loint(v), src_lane);
    const int hi = __builtin_amdgcn_readlane(__double2hiint(v), src_lane);
    return __hiloint2double(hi, lo);
}

template <int CTRL>
__device__ inline double dpp_from(double v)   // the value of the lane that CTRL selects
{
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xF, 0xF, false);
    return __hiloint2double(hi, lo);
}

// upper half of a <-> lower half of b (HALF = 32), or the odd 16-lane rows of a <-> the even ones of b
template <int HALF>
__device__ inline void lane_swap(double &a, double &b)
{
    const auto lo = HALF == 32 ? __builtin_amdgcn_permlane32_swap(__double2loint(a), __double2loint(b), false, false)
                               : __builtin_amdgcn_permlane16_swap(__double2loint(a), __double2loint(b), false, false);
    const auto hi = HALF == 32 ? __builtin_amdgcn_permlane32_swap(__double2hiint(a), __double2hiint(b), false, false)
                               : __builtin_amdgcn_permlane16_swap(__double2hiint(a), __double2hiint(b), false, false);
    a = __hiloint2double(hi[0], lo[0]);
    b = __hiloint2double(hi[1], lo[1]);
}

// One step of a cross-lane sum of doubles through the DPP data path (no LDS):
// adds to every lane the value of the lane that `CTRL` selects; lanes of rows
// outside ROW_MASK add zero.  With a full row mask every lane receives a value,
// so the destination needs no initial value.
template <int CTRL, int ROW_MASK>
__device__ inline double dpp_add(double v)
{
    const int lo = __double2loint(v), hi = __double2hiint(v);
    int plo, phi;
    if (ROW_MASK == 0xF) {
        plo = __builtin_amdgcn_mov_dpp(lo, CTRL, 0xF, 0xF, false);
        phi = __builtin_amdgcn_mov_dpp(hi, CTRL, 0xF, 0xF, false);
    } else {
        plo = __builtin_amdgcn_update_dpp(0, lo, CTRL, ROW_MASK, 0xF, false);
        phi = __builtin_amdgcn_update_dpp(0, hi, CTRL, ROW_MASK, 0xF, false);
    }
    return v + __hiloint2double(phi, plo);
}

// Sum over the 64 lanes of a wavefront in a fixed order; every lane gets the result.
__device__ inline double wave_sum(double v)
{
    v = dpp_add<0xB1, 0xF>(v);   // quad_perm [1,0,3,2]
    v = dpp_add<0x4E, 0xF>(v);   // quad_perm [2,3,0,1]
    v = dpp_add<0x141, 0xF>(v);  // row_half_mirror
    v = dpp_add<0x140, 0xF>(v);  // row_mirror: every lane of a 16-lane row holds the row's sum
    v = dpp_add<0x142, 0xA>(v);  // row_bcast15 into rows 1 and 3
    v = dpp_add<0x143, 0xC>(v);  // row_bcast31 into rows 2 and 3: lane 63 holds the total
    return lane_value(v, 63);
}

template <int CTRL, int ROW_MASK>
__device__ inline double dpp_max(double v)
{
    const int lo = __double2loint(v), hi = __double2hiint(v);
    // lanes outside ROW_MASK receive their own value back
    const int plo = __builtin_amdgcn_update_dpp(lo, lo, CTRL, ROW_MASK, 0xF, false);
    const int phi = __builtin_amdgcn_update_dpp(hi, hi, CTRL, ROW_MASK, 0xF, false);
    return fmax(v, __hiloint2double(phi, plo));
}

// Sum over a row of 16 lanes; every lane of the row gets the result.
__device__ inline double row_sum(double v)
{
    v = dpp_add<0xB1, 0xF>(v);
    v = dpp_add<0x4E, 0xF>(v);
    v = dpp_add<0x141, 0xF>(v);
    return dpp_add<0x140, 0xF>(v);
}

// Sum over a half-wavefront; every lane of the half gets the result.
__device__ inline double half_sum(double v)
{
    v = row_sum(v);
    double w = v;
    lane_swap<16>(v, w);
    return v + w;
}

// Maximum over the 64 lanes of a wavefront; every lane gets the result.
__device__ inline double wave_max(double v)
{
    v = dpp_max<0xB1, 0xF>(v);
    v = dpp_max<0x4E, 0xF>(v);
    v = dpp_max<0x141, 0xF>(v);
    v = dpp_max<0x140, 0xF>(v);
    v = dpp_max<0x142, 0xA>(v);
    v = dpp_max<0x143, 0xC>(v);
    return lane_value(v, 63);
}

// Maximum over a row of 16 lanes; every lane of the row gets the result.
__device__ inline double row_max(double v)
{
    v = dpp_max<0xB1, 0xF>(v);
    v = dpp_max<0x4E, 0xF>(v);
    v = dpp_max<0x141, 0xF>(v);
    return dpp_max<0x140, 0xF>(v);
}

// Maximum over a half-wavefront; every lane of the half gets the result.
__device__ inline double half_max(double v)
{
    v = row_max(v);
    double w = v;
    lane_swap<16>(v, w);
    return fmax(v, w);
}

// natural log of a positive finite double: exponent taken out exactly, the
// mantissa's log in single precision (absolute error about 5e-8)
__device__ inline double fast_log(double x)
{
    int e;
    double mant = frexp(x, &e);
    return (double)__logf((float)mant) + (double)e * 0.69314718055994530942;
}

// One term of a log-sum-exp with a running maximum.
__device__ inline void lse_step(double t, double &mx, double &sm)
{
    if (t > -INFINITY) {
        const double d = t - mx;
        const double e = (double)__expf(-fabsf((float)d));
        if (d > 0.0) {
            sm = fma(sm, e, 1.0);
            mx = t;
        } else {
            sm += e;
        }
    }
}

__device__ inline double fast_rcp(double x)   // 1 / x for a positive finite x, to about one unit in the last place
{
    double r = __builtin_amdgcn_rcp(x);
    r = fma(fma(-x, r, 1.0), r, r);
    r = fma(fma(-x, r, 1.0), r, r);
    return r;
}

// One step of the cross-lane sum of two values: lanes in the upper half (HALF = 32) or in the odd 16-lane
// rows (HALF = 16) end up with b's sum over the pair of lanes, the others with a's.
template <int HALF>
__device__ inline double halve(double a, double b)
{
    lane_swap<HALF>(a, b);
    return a + b;
}

// Sums of NV (4 or 8) values over the 64 lanes; lane l receives the sum of value l / (64 / NV).
template <int NV>
__device__ inline double reduce_values(double (&v)[NV])
{
    double s;
    if constexpr (NV == 4) {
        const double a = halve<32>(v[0], v[2]), b = halve<32>(v[1], v[3]);
        s = halve<16>(a, b);
    } else {
        const double a = halve<32>(v[0], v[4]), b = halve<32>(v[1], v[5]), c = halve<32>(v[2], v[6]),
                     d = halve<32>(v[3], v[7]);
        const double e = halve<16>(a, c), f = halve<16>(b, d);
        const bool odd = threadIdx.x & 8;
        const double keep = odd ? f : e, give = odd ? e : f;
        s = keep + dpp_from<0x128>(give);   // row_ror:8
    }
    s += dpp_from<0xB1>(s);    // quad_perm [1,0,3,2]
    s += dpp_from<0x4E>(s);    // quad_perm [2,3,0,1]
    s += dpp_from<0x141>(s);   // row_half_mirror
    if constexpr (NV == 4) s += dpp_from<0x140>(s);   // row_mirror
    return s;
}

// Factor row of lp = 64 T entries held by a wave: per 256 entries one 16-byte load of four consecutive entries
// per lane, then one 8-byte load if 128 or more are left, then one of 4 bytes.
template <int T>
struct FRow {
    static constexpr int Q4 = T / 4 * 4;
    float f[T];
    __device__ inline void load(const float *__restrict__ F, long long row, int lp, int lane)
    {
        F += row * lp;
#pragma unroll
        for (int q = 0; q < T / 4; ++q) {
            const float4 v = *(const float4 *)(F + (unsigned)(256 * q + 4 * lane));
            f[4 * q + 0] = v.x;
            f[4 * q + 1] = v.y;
            f[4 * q + 2] = v.z;
            f[4 * q + 3] = v.w;
        }
        if constexpr (T % 4 >= 2) {
            const float2 v = *(const float2 *)(F + (unsigned)(64 * Q4 + 2 * lane));
            f[Q4] = v.x;
            f[Q4 + 1] = v.y;
        }
        if constexpr (T % 2 == 1) f[T - 1] = F[(unsigned)(64 * (T - 1) + lane)];
    }
    // index into the length-lp vectors of register slot e
    __device__ static inline int kidx(int e, int lane)
    {
        if (e < Q4) return 256 * (e / 4) + 4 * lane + (e % 4);
        if (T % 4 >= 2 && e < Q4 + 2) return 64 * Q4 + 2 * lane + (e - Q4);
        return 64 * (T - 1) + lane;
    }
};

// Up to so many hash rounds RR is the number of rounds; ANY_ROUNDS stands for more of them.
constexpr int EXACT_ROUNDS = 4, ANY_ROUNDS = 8;

// The rounds' segments of a row's record, read from the packed metadata (wave-uniform: scalar registers).
template <int RR>
struct RecordWalk {
    unsigned shift[RR];  // entry e of round r stands at place e + shift[r] of the gathered vector
    int end[RR];         // ... and is below end[r]; rounds that do not exist are empty
};

// More rounds: the words shift and end of every round, a word per lane.  Held in scalars and compared one after the other,
// eight rounds cost more instructions per entry than everything else, and five rows of them more scalar registers
// than there are.
template <>
struct RecordWalk<ANY_ROUNDS> {
    int words;   // lane 2 r: shift[r], lane 2 r + 1: end[r]
};

template <int RR>
__device__ inline int record_total(const RecordWalk<RR> &W, int R)
{
    if constexpr (RR == ANY_ROUNDS)
        return __builtin_amdgcn_readlane(W.words, 2 * R - 1);
    else
        return W.end[RR - 1];
}

// Where entry e of the record gathers from; `zero_slot` past its end.
template <int RR, class Walk>
__device__ inline unsigned gather_place(const Walk &M, int e, unsigned zero_slot)
{
    // (readfirstlane: uniform already; a plain select of two members would become a load through a selected
    // address and keep the record in scratch memory)
    unsigned sh = __builtin_amdgcn_readfirstlane(M.shift[0]);
#pragma unroll
    for (int r = 1; r < RR; ++r) {
        const unsigned other = __builtin_amdgcn_readfirstlane(M.shift[r]);
        sh = e >= M.end[r - 1] ? other : sh;
    }
    return e < M.end[RR - 1] ? (unsigned)e + sh : zero_slot;
}

// Walks a record a chunk of 64 entries after the other, in ascending order: where entry e = c + lane of the chunk that
// starts at c gathers from, `other` past the record's end.
template <int RR>
struct RecordCursor {
    const RecordWalk<RR> &W;
    __device__ inline RecordCursor(const RecordWalk<RR> &walk, int) : W(walk) {}
    __device__ inline unsigned place(int, int e, unsigned other) { return gather_place<RR>(W, e, other); }
};

// The round that the chunk begins in is at hand, the next ones are taken up where they begin: a comparison per round that
// ends in the chunk, not one per round there is.
template <>
struct RecordCursor<ANY_ROUNDS> {
    const int words, R, total;
    int r, end;
    unsigned shift;
    __device__ inline RecordCursor(const RecordWalk<ANY_ROUNDS> &walk, int rounds)
        : words(walk.words), R(rounds), total(record_total<ANY_ROUNDS>(walk, rounds)), r(0),
          end(__builtin_amdgcn_readlane(walk.words, 1)), shift((unsigned)__builtin_amdgcn_readlane(walk.words, 0))
    {
    }
    __device__ inline unsigned place(int c, int e, unsigned other)
    {
        unsigned sh = shift;
        while (end < c + 64 && r + 1 < R) {   // uniform
            const int before = end;
            ++r;
            shift = (unsigned)__builtin_amdgcn_readlane(words, 2 * r);
            end = __builtin_amdgcn_readlane(words, 2 * r + 1);
            sh = e >= before ? shift : sh;
        }
        return e < total ? (unsigned)e + sh : other;
    }
};

// the records are written once at build time: reading them through the constant
// address space lets the compiler use scalar loads although the kernel also stores
typedef const __attribute__((address_space(4))) int *const_int_ptr;

__device__ inline long long record_base(const PassSide &S, long long row)
{
    const_int_ptr rec = (const_int_ptr)(S.meta + row * S.meta_stride);
    return ((long long)rec[1] << 32) | (unsigned)rec[0];
}

// (an empty record for a row past the last one)
template <int RR>
__device__ inline void load_walk(RecordWalk<RR> &W, const PassSide &S, int R, long long row)
{
    const bool exists = row < S.rows;
    const int *at = S.meta + (exists ? row : S.rows - 1) * S.meta_stride;
    if constexpr (RR == ANY_ROUNDS) {
        const int lane = threadIdx.x & 63, word = at[6 + (lane < 2 * R ? lane : 0)];
        W.words = exists ? word : 0;
    } else {
        const_int_ptr rec = (const_int_ptr)at;
#pragma unroll
        for (int r = 0; r < RR; ++r) {
            W.shift[r] = (unsigned)rec[6 + 2 * r];
            const int end = rec[7 + 2 * r];
            W.end[r] = !exists ? 0 : end;
        }
    }
}

// Per-row metadata, read from the packed record (see meta_kernel): wave-uniform,
// so it lives in scalar registers.
template <int RR>
struct RowMeta {
    long long base;
    float marg;
    double log_marg;
    RecordWalk<RR> walk;
    int pos;     // lane r < R: position of the row in round r's bucket order
    double lin;  // query mode: the row's current scaling
};

template <int RR, int MODE>
__device__ inline void load_meta(RowMeta<RR> &M, const PassSide &S, int R, long long row, int lane)
{
    const_int_ptr rec = (const_int_ptr)(S.meta + row * S.meta_stride);
    M.base = ((long long)rec[1] << 32) | (unsigned)rec[0];
    M.marg = __int_as_float(rec[2]);
    M.log_marg = __hiloint2double(rec[5], rec[4]);
    load_walk<RR>(M.walk, S, R, row);
    M.pos = (MODE != PASS_QUERY && lane < R) ? rec[6 + 2 * R + lane] : 0;
    M.lin = MODE == PASS_QUERY ? S.lin_out[row] : 0.0;
}

// A sweep that finishes the previous sweep's reduction itself passes the totals
// from the reducing workgroups to all others through the accumulator itself:
// the sweep before filled the accumulator with ACC_PENDING (a NaN bit pattern no
// arithmetic produces), the reducing workgroups overwrite it with device-scope
// stores, and a reader simply re-reads (device scope) until no entry is pending.
// No flag and no fence is involved, so a hand-over costs one store and one load
// through memory.
constexpr unsigned long long ACC_PENDING = 0x7FF8A5A55A5AC3C3ull;

struct FuseArgs {
    const double *prev_partial;  // [prev_groups][lp + 3] partial sums the previous sweep left
    int prev_groups;
    int direct;                  // every workgroup takes the totals for itself
    double *acc;                 // where the totals go: this sweep's input accumulator (lp + 2 entries)
    const double *shift_other;   // exponent of the other side's vector (the previous sweep's own)
    double *shift_next;          // the exponent of the other side's next vector
    const double *shift_self;    // exponent of this side's vector
    double *mark_pending;        // accumulator the NEXT sweep reduces into (nullable): filled with ACC_PENDING
    unsigned long long *timeouts;
    unsigned long long wait_ticks;  // how long a workgroup re-reads pending totals before it gives up (100 MHz clock)
};

// Marks the accumulator that the next sweep will fill as pending (one wavefront of
// one workgroup; ordinary stores, visible to the next launch).
__device__ inline void mark_pending(const FuseArgs &Fz, int lp)
{
    if (Fz.mark_pending && blockIdx.x == gridDim.x - 1 && threadIdx.x < 64)
        for (int k = threadIdx.x; k <= lp + 1; k += 64) ((unsigned long long *)Fz.mark_pending)[k] = ACC_PENDING;
}

// The total of a column of the partial sums is taken in one fixed order everywhere, whoever takes it: row g belongs
// to running sum g % 64; the four of them with the same g % 16 are added up in turn, then four such sums 4 q .. 4 q + 3
// in turn, and the four results as (0 + 2) + (1 + 3).  The last column's total is a maximum.
constexpr int REDUCE_COLUMNS = 16;
__device__ inline double join_sums(bool is_max, double a, double b) { return is_max ? fmax(a, b) : a + b; }

// By one workgroup of 1024 threads for 16 columns: lane l of wavefront w has row 4 w + l / 16 and every 64th after it,
// 256 rows being four loads per lane.  Column 16 b + l % 16 is returned in lanes 0 .. 15 of wavefront 0.  red: [64][16]
// doubles of LDS.  (64 columns per workgroup, 16 loads per lane: a compute unit then has to bring in 131 KB by itself,
// and the totals of 259 columns were there 3.3 us after the start of the sweep instead of 2.5.)
__device__ inline double reduce_columns(const double *__restrict__ partial, int groups, int stride, int b, int max_column,
                                        double *red)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int col = lane & 15, sub = lane >> 4, k = REDUCE_COLUMNS * b + col;
    const bool is_max = k == max_column;
    const double none = is_max ? -INFINITY : 0.0;
    double s = none;
    if (k < stride) {
#pragma unroll 4
        for (int g = 4 * wave + sub; g < groups; g += 64) s = join_sums(is_max, s, partial[(long long)g * stride + k]);
    }
    red[(4 * wave + sub) * 16 + col] = s;
    __syncthreads();
    s = none;
    if (wave == 0) {
#pragma unroll
        for (int w = 4 * sub; w < 4 * sub + 4; ++w) {
            double r = red[w * 16 + col];
#pragma unroll
            for (int q = 1; q < 4; ++q) r = join_sums(is_max, r, red[(w + 16 * q) * 16 + col]);
            s = w == 4 * sub ? r : join_sums(is_max, s, r);
        }
        double o = s;
        lane_swap<32>(s, o);
        s = join_sums(is_max, s, o);
        o = s;
        lane_swap<16>(s, o);
        s = join_sums(is_max, s, o);
    }
    return s;
}

// The totals of the previous sweep's partial sums (bitwise those of reduce_partials_kernel), 16 columns per
// workgroup, published with device-scope stores by the first workgroups of the grid (in turns if it has fewer
// than there are columns for).  Nothing here waits, so a reducing workgroup always gets through.
// (With the partial sums requested first and added up only after the workgroup's rows had been requested a sweep
// is slower, 15.8 against 13.7 us at 20 000 rows of 256 entries: loads return in order, so everybody's totals then
// wait for those rows.)
__device__ inline void reduce_publish(const FuseArgs &Fz, int lp, double *red)
{
    const int stride = lp + 3, blocks = (stride + REDUCE_COLUMNS - 1) / REDUCE_COLUMNS;
    for (int b = blockIdx.x; b < blocks; b += gridDim.x) {
        // what the last column needs besides is requested with the sums: the exponent the previous sweep's vector
        // was stored with, and this side's
        const double m_in = *Fz.shift_other, m_self = *Fz.shift_self;
        if (b != (int)blockIdx.x) __syncthreads();   // the previous turn has read the sums
        const double s = reduce_columns(Fz.prev_partial, Fz.prev_groups, stride, b, lp + 2, red);
        const int k = REDUCE_COLUMNS * b + threadIdx.x;
        if (threadIdx.x < REDUCE_COLUMNS && k < stride) {
            if (k < lp) {
                __hip_atomic_store(Fz.acc + k, s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            } else if (k == lp + 2) {
                // ... and the factor exp(-m_in - m_self) this sweep applies to its results
                __hip_atomic_store(Fz.acc + lp, m_in, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_store(Fz.acc + lp + 1, exp(-m_in - m_self), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                *Fz.shift_next = (s > -INFINITY && s < INFINITY) ? s : 0.0;
            }
        }
    }
}

// Up to 64 factor columns and 64 partial sums: every workgroup takes the totals for itself (at most 34 KB from the
// cache) and nothing has to be handed over: a store, a trip through memory and the wait for it less per sweep (1024
// rows: 5.5 us instead of 6.2).  With 256 partial sums, 137 KB, it is the slower way (50 000 rows: 8.9 against 8.5).
// Wavefront w has the rows g % 16 == w, a lane a column; all loads are requested at once, before the workgroup's own
// rows are.  The exponents exist twice (shift_other is read by every workgroup, shift_next written by one).
constexpr int DIRECT_GROUPS = 64;
struct DirectTotals {
    double v[4], top, m_in, m_self;
    __device__ inline void request(const FuseArgs &Fz, int lp)
    {
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, stride = lp + 3, last = Fz.prev_groups - 1;
        m_in = *Fz.shift_other;
        m_self = *Fz.shift_self;
        const double *__restrict__ at = Fz.prev_partial + lane;
        // (a row past the last one repeats it and is not added)
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = at[(wave + 16 * u < last ? wave + 16 * u : last) * stride];
        // (the first wavefront: a row per lane)
        top = wave == 0 ? Fz.prev_partial[(lane < last ? lane : last) * stride + lp + 2] : -INFINITY;
    }
    // the total of column `lane` (lp = 64); red: [16][64] doubles of LDS
    __device__ inline double finish(const FuseArgs &Fz, int lp, double *red, double &m_in_out, double &e_out)
    {
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
        double r = wave < Fz.prev_groups ? v[0] : 0.0;
#pragma unroll
        for (int q = 1; q < 4; ++q) r += wave + 16 * q < Fz.prev_groups ? v[q] : 0.0;
        red[wave * 64 + lane] = r;
        m_in_out = m_in;
        e_out = exp(-m_in - m_self);   // the factor this sweep applies to its results
        __syncthreads();
        double p[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            p[q] = red[4 * q * 64 + lane];
#pragma unroll
            for (int j = 1; j < 4; ++j) p[q] += red[(4 * q + j) * 64 + lane];
        }
        const double s = (p[0] + p[2]) + (p[1] + p[3]);
        if (blockIdx.x == 0 && wave == 0) {   // for queries and derivatives after the run, and for the next sweep
            Fz.acc[lane] = s;
            if (lane == 0) {
                Fz.acc[lp] = m_in;
                Fz.acc[lp + 1] = e_out;
            }
            const double m = wave_max(top);
            if (lane == 0) *Fz.shift_next = (m > -INFINITY && m < INFINITY) ? m : 0.0;
        }
        return s;
    }
};

// Reads the totals (lp + 2 doubles) into `ysh`, re-reading until the reducing
// workgroups of this launch have replaced every pending entry (bounded wait).
// Called by one wavefront of every workgroup; the caller synchronises the
// workgroup afterwards.
__device__ inline void fused_fetch(const FuseArgs &Fz, const double *acc, int lp, double *ysh)
{
    const int lane = threadIdx.x & 63;
    const unsigned long long *src = (const unsigned long long *)acc;
    // once a wait has timed out no later wait is attempted (the run is reported as failed)
    bool give_up = __hip_atomic_load(Fz.timeouts, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0ull;
    const unsigned long long t0 = wall_clock64();
    for (;;) {
        bool pending = false;
        for (int k = lane; k <= lp + 1; k += 64) {
            const unsigned long long v = __hip_atomic_load(src + k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            pending |= v == ACC_PENDING;
            ((unsigned long long *)ysh)[k] = v;
        }
        if (!__any(pending) || give_up) break;
        if (wall_clock64() - t0 > Fz.wait_ticks) {
            if (lane == 0) atomicAdd(Fz.timeouts, 1ull);
            give_up = true;
        }
    }
}

// The totals into every wavefront's registers, by whichever of the two ways (the workgroup's row requests stand
// between the request of the partial sums and this).
template <int T>
__device__ inline void take_totals(const FuseArgs &Fz, const double *acc_in, int lp, double *ysh, DirectTotals &totals,
                                   double (&yreg)[T], double &m_in, double &e_out)
{
    const int lane = threadIdx.x & 63;
    if (T == 1 && Fz.direct) {
        yreg[0] = totals.finish(Fz, lp, ysh + lp + 2, m_in, e_out);
    } else {
        if (threadIdx.x < 64) fused_fetch(Fz, acc_in, lp, ysh);
        __syncthreads();
        m_in = ysh[lp];
        e_out = ysh[lp + 1];
#pragma unroll
        for (int t = 0; t < T; ++t) yreg[t] = ysh[FRow<T>::kidx(t, lane)];
    }
}

// End of a sweep: the sums over the workgroup's wavefronts (upper half of the waves hands its values to the
// lower half first) as one partial per workgroup.  zsh: [PASS_WAVES / 2][lp + 3].
template <int T>
__device__ inline void group_partials(const double (&zacc)[T], double q0, double q1, double maxlog, int lp, double *zsh,
                                      double *partial)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int stride = lp + 3;
    constexpr int HALF = PASS_WAVES / 2;
    double *mine = zsh + (wave % HALF) * stride;
    if (wave >= HALF) {
#pragma unroll
        for (int t = 0; t < T; ++t) mine[FRow<T>::kidx(t, lane)] = zacc[t];
        if (lane == 0) {
            mine[lp] = q0;
            mine[lp + 1] = q1;
            mine[lp + 2] = maxlog;
        }
    }
    __syncthreads();
    if (wave < HALF) {
#pragma unroll
        for (int t = 0; t < T; ++t) mine[FRow<T>::kidx(t, lane)] += zacc[t];
        if (lane == 0) {
            mine[lp] += q0;
            mine[lp + 1] += q1;
            mine[lp + 2] = fmax(mine[lp + 2], maxlog);
        }
    }
    __syncthreads();
    for (int k = threadIdx.x; k < stride; k += PASS_THREADS) {
        double s = k == lp + 2 ? -INFINITY : 0.0;
#pragma unroll
        for (int w = 0; w < HALF; ++w) s = k == lp + 2 ? fmax(s, zsh[w * stride + k]) : s + zsh[w * stride + k];
        partial[(long long)blockIdx.x * stride + k] = s;
    }
}

inline size_t pass_lds_bytes(int lp, bool fused)
{
    size_t doubles = (size_t)(PASS_WAVES / 2) * (lp + 3);
    if (fused) doubles += (size_t)lp + 2 + 64 * REDUCE_COLUMNS;
    return sizeof(double) * doubles;
}

// sweeps with a sparse part by the length of the factor rows: up to 128 entries, up to 256, more
hipError_t launch_short_sweep(const PassSide &S, const Handle &h, int mode, const FuseArgs &F, bool fused_in, int groups,
                              double *partial, unsigned long long *cnt, hipStream_t s);
hipError_t launch_mid_sweep(const PassSide &S, const Handle &h, int mode, const FuseArgs &F, bool fused_in, int groups,
                            double *partial, unsigned long long *cnt, hipStream_t s);
hipError_t launch_long_sweep(const PassSide &S, const Handle &h, int mode, const FuseArgs &F, bool fused_in, int groups,
                             double *partial, unsigned long long *cnt, hipStream_t s);
int rows_at_a_time(const Handle &h, long long rows);

// sweeps without a sparse part (kernels_nystrom.hip), and how many workgroups (partial sums) one has
hipError_t launch_nystrom_pass(const PassSide &S, const Handle &h, int mode, const FuseArgs *fuse, bool fused_in,
                               double *partial, unsigned long long *cnt, hipStream_t s);
int nystrom_sweep_groups(const Handle &h, long long rows);

}  // namespace lcn
