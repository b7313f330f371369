// The Sinkhorn half-iteration on the Nystrom kernel alone (no hash rounds, Sec. 4): for every row i of one side
//     s_i = F_i . acc_in,   out_i = marg_i / s_i,   acc_out = F^T out
// with F = U, acc_in = y = W v, acc_out = z = U^T u for the rows of X and F = W^T, acc_in = z, acc_out = y
// for the rows of Y.  State, exponents and hand-over of the totals as in the sweep with a sparse part
// (sweep.h); what differs is how rows are dealt out.
//
// One wavefront owns RG consecutive rows at a time: their factor rows are one contiguous piece of memory and are
// requested together, the RG partial sums go through the cross-lane reduction together (recursive halving:
// each step halves the number of values a lane holds), and what is done once per row -- reciprocal,
// logarithm, stores -- is done for the RG rows at once, a row per group of lanes.  With a row at a time a short
// factor row (64 entries: one load) costs over a hundred instructions and a trip to memory of its own;
// what bounds the sweep now is the launch, the hand-over and one trip to memory.  50 000 rows of 64
// entries: 22.9 -> 8.4 us per sweep.  Rows with a sparse part are dealt in groups too (sweep.h), but in smaller ones: their
// records take registers and the wavefronts are needed to hide the walk over them.
#include "iter_common.h"

namespace lcn {

template <int T, int MODE, bool FUSED, int RG>
__global__ __launch_bounds__(PASS_THREADS) void nystrom_pass_kernel(PassSide S, int lp, double *partial,
                                                                    unsigned long long *counters, FuseArgs Fz)
{
    constexpr int NV = RG <= 4 ? 4 : 8;
    constexpr int GL = 64 / NV;      // lanes per row once the sums are taken
    extern __shared__ double zsh[];  // [PASS_WAVES / 2][lp + 3], then [lp + 2] and [16][64] if FUSED
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int groups = (int)((S.rows + RG - 1) / RG), nwaves = (int)gridDim.x * PASS_WAVES;
    // dealt out from the last workgroup down: the reducing workgroups of a fused sweep start late
    int g = ((int)gridDim.x - 1 - (int)blockIdx.x) * PASS_WAVES + wave;
    const int stride = lp + 3;
    double *ysh = zsh + (size_t)(PASS_WAVES / 2) * stride;
    if (MODE == PASS_UPDATE) mark_pending(Fz, lp);
    DirectTotals totals;
    if (FUSED && T == 1 && Fz.direct)
        totals.request(Fz, lp);
    else if (FUSED)
        reduce_publish(Fz, lp, ysh + lp + 2);
    const double m_self = MODE == PASS_QUERY ? S.acc_out[lp] : *S.shift_self;
    double m_in = 0.0, e_out = 1.0;
    double maxlog = -INFINITY, q0 = 0.0, q1 = 0.0;
    double yreg[T], zacc[T];
#pragma unroll
    for (int t = 0; t < T; ++t) yreg[t] = zacc[t] = 0.0;
    unsigned nonpos = 0;
    // this lane's row of a group once the sums are taken, and its number among the lanes of that row
    const int my = lane / GL, sub = lane % GL;

    FRow<T> f[RG];
    float marg;             // of this lane's row
    double log_marg, lin;   // (PASS_INIT: log_marg holds the row's log scaling)
    auto request = [&]() {  // rows past the last one repeat it and are dropped
        const long long row0 = (long long)g * RG;
#pragma unroll
        for (int t = 0; t < RG; ++t) f[t].load(S.F, row0 + t < S.rows ? row0 + t : S.rows - 1, lp, lane);
        const long long mine = row0 + my < S.rows ? row0 + my : S.rows - 1;
        const int *rec = S.meta + mine * S.meta_stride;
        marg = __int_as_float(rec[2]);
        log_marg = MODE == PASS_INIT ? (double)S.log_out[mine] : __hiloint2double(rec[5], rec[4]);
        lin = MODE == PASS_QUERY ? S.lin_out[mine] : 0.0;
    };
    // (unconditional, so that the loads in flight can be counted: a wavefront without rows requests the last group)
    const bool busy = g < groups;
    if (!busy) g = groups - 1;
    request();
    if (FUSED) {
        take_totals<T>(Fz, S.acc_in, lp, ysh, totals, yreg, m_in, e_out);
    } else if (MODE != PASS_INIT) {
        m_in = S.acc_in[lp];
        e_out = MODE == PASS_UPDATE ? exp(-m_in - m_self) : exp(m_in + m_self);
#pragma unroll
        for (int t = 0; t < T; ++t) yreg[t] = S.acc_in[FRow<T>::kidx(t, lane)];
    }
    if (busy) for (;;) {
        const long long mine = (long long)g * RG + my;
        const bool exists = my < RG && mine < S.rows;
        double out;
        if (MODE == PASS_INIT) {
            out = exists ? exp(log_marg - m_self) : 0.0;
            if (exists && log_marg > maxlog && log_marg < INFINITY) maxlog = log_marg;
        } else {
            double acc[NV];
#pragma unroll
            for (int t = 0; t < NV; ++t) acc[t] = 0.0;
#pragma unroll
            for (int k = 0; k < T; ++k)
#pragma unroll
                for (int t = 0; t < RG; ++t) acc[t] = fma((double)f[t].f[k], yreg[k], acc[t]);
            if (MODE == PASS_UPDATE) {
                // the entries stay in registers as floats: without this the compiler keeps the converted
                // doubles, twice the registers, from here to the accumulation below
#pragma unroll
                for (int t = 0; t < RG; ++t)
#pragma unroll
                    for (int k = 0; k < T; ++k) asm("" : "+v"(f[t].f[k]));
            }
            const double s = reduce_values<NV>(acc);
            if (MODE == PASS_UPDATE) {
                float lo;
                if (s > 0.0) {
                    out = (double)marg * fast_rcp(s) * e_out;
                    const double lg = log_marg - fast_log(s) - m_in;
                    lo = (float)lg;
                    maxlog = exists ? fmax(maxlog, lg) : maxlog;
                } else {
                    out = NAN;
                    lo = NAN;
                    if (exists && sub == 0) ++nonpos;
                }
                if (!exists) out = 0.0;
                if (exists && sub == 0) S.log_out[mine] = lo;
            } else {  // PASS_QUERY
                out = lin;
                const double ri = out * s * e_out;
                if (exists && sub == 0) {
                    if (S.marg_out) S.marg_out[mine] = (float)ri;
                    if (out > 0.0) q0 += ri * (log(out) + m_self);
                    q1 += fabs(ri - (double)marg);
                }
            }
        }
        if (MODE != PASS_QUERY) {
            if (exists && sub == 0) S.lin_out[mine] = out;
#pragma unroll
            for (int t = 0; t < RG; ++t) {
                const double o = lane_value(out, t * GL);
#pragma unroll
                for (int k = 0; k < T; ++k) zacc[k] = fma((double)f[t].f[k], o, zacc[k]);
            }
        }
        g += nwaves;
        if (g >= groups) break;
        request();
    }

    if (MODE == PASS_QUERY) {
        q0 = wave_sum(q0);
        q1 = wave_sum(q1);
    } else {
        maxlog = wave_max(maxlog);
    }
    group_partials<T>(zacc, q0, q1, maxlog, lp, zsh, partial);
    if (nonpos) atomicAdd(&counters[0], (unsigned long long)nonpos);
}

// Rows a wavefront takes at a time: eight, or as many as its registers hold of long rows; fewer if that
// takes fewer rounds times rows (a side too small to give every wavefront eight rows).
static int rows_per_wave(const Handle &h, long long rows)
{
    if (h.lp > 256) return 4;
    const long long waves = (long long)h.grid * PASS_WAVES;
    const long long r4 = ((rows + 3) / 4 + waves - 1) / waves * 4, r8 = ((rows + 7) / 8 + waves - 1) / waves * 8;
    return r4 < r8 ? 4 : 8;
}

int nystrom_sweep_groups(const Handle &h, long long rows)
{
    const long long per = (long long)PASS_WAVES * rows_per_wave(h, rows), g = (rows + per - 1) / per;
    return (int)(g < h.grid ? g : h.grid);
}

template <int T, int RG>
static void launch_nystrom_rows(const PassSide &S, const Handle &h, int mode, const FuseArgs *fuse, bool fused_in,
                                double *partial, unsigned long long *cnt, int grid, hipStream_t s)
{
    const FuseArgs F = fuse ? *fuse : FuseArgs{};
    const dim3 g(grid), b(PASS_THREADS);
    const size_t lds = pass_lds_bytes(h.lp, fused_in);
    if (mode == PASS_UPDATE && fused_in)
        hipLaunchKernelGGL((nystrom_pass_kernel<T, PASS_UPDATE, true, RG>), g, b, lds, s, S, h.lp, partial, cnt, F);
    else if (mode == PASS_UPDATE)
        hipLaunchKernelGGL((nystrom_pass_kernel<T, PASS_UPDATE, false, RG>), g, b, lds, s, S, h.lp, partial, cnt, F);
    else if (mode == PASS_QUERY)
        hipLaunchKernelGGL((nystrom_pass_kernel<T, PASS_QUERY, false, RG>), g, b, lds, s, S, h.lp, partial, cnt, F);
    else
        hipLaunchKernelGGL((nystrom_pass_kernel<T, PASS_INIT, false, RG>), g, b, lds, s, S, h.lp, partial, cnt, F);
}

hipError_t launch_nystrom_pass(const PassSide &S, const Handle &h, int mode, const FuseArgs *fuse, bool fused_in,
                               double *partial, unsigned long long *cnt, hipStream_t s)
{
    const int grid = nystrom_sweep_groups(h, S.rows), rg = rows_per_wave(h, S.rows);
#define LCN_NYS(T_)                                                                                                    \
    case T_:                                                                                                           \
        if (T_ <= 4 && rg == 8)                                                                                        \
            launch_nystrom_rows<(T_ <= 4 ? T_ : 1), 8>(S, h, mode, fuse, fused_in, partial, cnt, grid, s);             \
        else                                                                                                           \
            launch_nystrom_rows<T_, 4>(S, h, mode, fuse, fused_in, partial, cnt, grid, s);                             \
        break
    switch (h.lp / 64) {
        LCN_NYS(1);
        LCN_NYS(2);
        LCN_NYS(3);
        LCN_NYS(4);
        LCN_NYS(5);
        LCN_NYS(6);
        LCN_NYS(7);
        LCN_NYS(8);
        default: return hipErrorInvalidValue;
    }
#undef LCN_NYS
    return hipGetLastError();
}

}  // namespace lcn
