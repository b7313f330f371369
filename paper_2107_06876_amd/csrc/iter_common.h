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

// Per-row metadata, read from the packed record (see meta_kernel): wave-uniform,
// so it lives in scalar registers.
template <int RR>
struct RowMeta {
    long long base;
    float marg;
    double log_marg;
    int vstart[RR];
    int len[RR];
    int pos;     // lane r < R: position of the row in round r's bucket order
    double lin;  // query mode: the row's current scaling
};

template <int RR, int MODE>
__device__ inline void load_meta(RowMeta<RR> &M, const PassSide &S, int R, long long row, int lane)
{
    // the records are written once at build time: reading them through the constant
    // address space lets the compiler use scalar loads although the kernel also stores
    typedef const __attribute__((address_space(4))) int *const_int_ptr;
    const_int_ptr rec = (const_int_ptr)(S.meta + row * S.meta_stride);
    M.base = ((long long)rec[1] << 32) | (unsigned)rec[0];
    M.marg = __int_as_float(rec[2]);
    M.log_marg = __hiloint2double(rec[5], rec[4]);
#pragma unroll
    for (int r = 0; r < RR; ++r) {
        M.vstart[r] = r < R ? rec[6 + 2 * r] : 0;
        M.len[r] = r < R ? rec[7 + 2 * r] : 0;
    }
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
    double *acc;                 // where the totals go: this sweep's input accumulator (lp + 2 entries)
    double *shift_other;         // exponent of the other side's vector (the previous sweep's own)
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

// The sum of the per-workgroup partials in the fixed order of
// reduce_partials_kernel (bitwise the same result), by workgroup `b` for its 64
// entries, published with device-scope stores.  Nothing here waits, so a
// reducing workgroup always gets through.
__device__ inline void reduce_publish(const FuseArgs &Fz, int b, int lp, double *red)
{
    double *acc = Fz.acc;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int nw = blockDim.x >> 6;
    const int stride = lp + 3;
    const int k = b * 64 + lane;
    const bool is_max = k == lp + 2;
    // 16 running sums as in reduce_partials_kernel (sum a takes partials a, a + 16, ...),
    // shared out among the wavefronts this workgroup has
    for (int a = wave; a < 16; a += nw) {
        double s = is_max ? -INFINITY : 0.0;
        if (k < stride) {
#pragma unroll 16
            for (int g = a; g < Fz.prev_groups; g += 16) {
                const double v = Fz.prev_partial[(long long)g * stride + k];
                s = is_max ? fmax(s, v) : s + v;
            }
        }
        red[a * 64 + lane] = s;
    }
    __syncthreads();
    if (wave == 0 && k < stride) {
        double s = is_max ? -INFINITY : 0.0;
#pragma unroll
        for (int w = 0; w < 16; ++w) s = is_max ? fmax(s, red[w * 64 + lane]) : s + red[w * 64 + lane];
        if (k < lp) {
            __hip_atomic_store(acc + k, s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        } else if (is_max) {
            // the exponent the previous sweep's vector was stored with, and the factor
            // exp(-m_in - m_self) this sweep applies to its results
            const double m_in = *Fz.shift_other;
            __hip_atomic_store(acc + lp, m_in, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(acc + lp + 1, exp(-m_in - *Fz.shift_self), __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
            *Fz.shift_other = (s > -INFINITY && s < INFINITY) ? s : 0.0;
        }
    }
}

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
    if (fused) doubles += (size_t)lp + 2 + 16 * 64;
    return sizeof(double) * doubles;
}

// sweeps without a sparse part (kernels_nystrom.hip), and how many workgroups (partial sums) one has
hipError_t launch_nystrom_pass(const PassSide &S, const Handle &h, int mode, const FuseArgs *fuse, bool fused_in,
                               double *partial, unsigned long long *cnt, hipStream_t s);
int nystrom_sweep_groups(const Handle &h, long long rows);

}  // namespace lcn
