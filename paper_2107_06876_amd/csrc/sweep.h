// The Sinkhorn half-iteration (Sec. 2 eq. 2 on the decomposed kernel of Sec. 4):
// for every row i of one side
//     s_i   = F_i . acc_in  +  (row record of sparse values) . (gathered scalings)
//     out_i = marg_i / s_i
// and, in the same sweep, acc_out = F^T out for the other side's next sweep.
// For the rows of X: F = U, acc_in = y = W v, acc_out = z = U^T u.
// For the rows of Y: F = W^T, acc_in = z, acc_out = y.
// Each stored value (factor entry or sparse value) is read exactly once per
// sweep.  Consecutive lanes read consecutive addresses of a factor row and of
// the row's record of sparse values; a wavefront works on several rows at a time.
//
// Log-domain stabilisation (App. "Implementational details"): the state is the
// natural log of each scaling (fp32, what is reported).  Because the Nystrom
// part and the correction have signed entries the kernel cannot itself be held
// as logs, so the largest exponent is taken out per vector instead: the working
// copy of a scaling vector is exp(log x - M) in fp64, with M the largest log of
// that vector one iteration earlier (any reference works; logs move slowly), and
// M travels with every quantity derived from the vector.  Products are
// accumulated in fp64.
#pragma once

#include "iter_common.h"

namespace lcn {

// FUSED (update sweeps after the first of a run): the previous sweep's partial
// sums have not been added up yet.  The first workgroups of
// this launch do that before their own rows and publish the totals; every
// workgroup requests its first rows, then waits for the totals (bounded wait;
// the reducing workgroups have the lowest indices, are dispatched first and
// wait for nothing, so the wait ends).  This saves a dependent kernel launch
// per sweep without any device-wide fence.
//
// RG rows per wavefront at a time, as in the sweep without a sparse part: the cross-lane sums, the reciprocal, the
// logarithm and the stores are then paid once for RG rows.
//
// A row's record is walked flat: its values of all rounds lie back to back, so 64 consecutive entries are one
// load whatever the rounds' lengths, and the entry's place in the gathered vector is its number plus an offset
// that changes where a round's segment ends (uniform comparisons).  V: entries of a row requested with it, in
// wavefronts; the rest of a longer record follows in trips of SWEEP_TRIP wavefronts.
template <int T, int RR, int RG, int V, int MODE, bool FUSED>
__global__ __launch_bounds__(PASS_THREADS) void pass_kernel(PassSide S, int R, int lp, double *partial,
                                                            unsigned long long *counters, FuseArgs Fz)
{
    constexpr int NV = RG <= 4 ? 4 : 8;
    constexpr int GL = 64 / NV;      // lanes per row once the sums are taken (at least 8: one per hash round)
    constexpr int TRIP = SWEEP_TRIP;
    static_assert(64 * TRIP <= VALUE_SLACK && 64 * V <= VALUE_SLACK, "read past the last record");
    extern __shared__ double zsh[];  // [PASS_WAVES / 2][lp + 3], then [lp + 2] and the reduction's scratch if FUSED
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int groups = (int)((S.rows + RG - 1) / RG), nwaves = (int)gridDim.x * PASS_WAVES;
    // Rows are dealt out from the last workgroup down: the reducing workgroups of a fused
    // sweep (the first few) start late, so they get the row slots that may hold one group less.
    // The dealing is the same with and without fusion, so both give the same bits.
    int g = ((int)gridDim.x - 1 - (int)blockIdx.x) * PASS_WAVES + wave;
    const int stride = lp + 3;
    double *ysh = zsh + (size_t)(PASS_WAVES / 2) * stride;
    // exponents taken out of this side's vector (m_self) and of the input vectors (m_in)
    // (a query reads the exponent its vector was stored with, kept beside the accumulator it produced)
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
    unsigned nonpos = 0, range = 0;
    // this lane's row of a group once the sums are taken, and its number among the lanes of that row
    const int my = lane / GL, sub = lane % GL;

    // The bucket-ordered copies of the scalings are single precision in this kernel (the buffers are
    // sized for doubles; the logarithmic kernels keep doubles there): they are gathered once per
    // stored value, and at half the size they stay in the per-die cache beside the streamed rows.
    // The exponent taken out keeps the largest entry near one, and the copies are stored times
    // PERM_SCALE = 2^64 (exact): single precision then holds entries from 2^-190 (e^-131) below the
    // vector's largest up to 2^63 (e^43) above it.  A sum's sparse part is scaled back before the
    // factor part is added.  An entry that grows past that within one iteration overflows its copy:
    // counted, and the run is reported as failed (LCN_ERR_RANGE).
    const float *__restrict__ perm_in = reinterpret_cast<const float *>(S.perm_in);
    float *__restrict__ perm_out = reinterpret_cast<float *>(S.perm_out);
    // Loads are issued for whole wavefront-wide chunks without predication: lanes
    // beyond a record's length read the next stored values (masked when used; the
    // arrays end with VALUE_SLACK entries, see record_reach.h) and the zero slot behind the gathered vector.
    const unsigned zero_slot = (unsigned)(R * S.rows_in);
    RecordWalk<RR> walk[RG];   // of the group at hand (scalars)
    long long base = 0;        // where the records of the group begin: they lie back to back
    FRow<T> f[RG];
    float tv[RG][V], pv[RG][V];
    float marg = 0.f;
    double log_marg = 0.0, lin = 0.0;   // of this lane's row (PASS_INIT: log_marg holds its log scaling)
    int pos = 0;                        // lane `sub` < R: position of the row in that round's bucket order
    auto load_walks = [&]() {
        if (MODE == PASS_INIT) return;
        const long long row0 = (long long)g * RG;
        base = record_base(S, row0);
#pragma unroll
        for (int t = 0; t < RG; ++t) load_walk<RR>(walk[t], S, R, row0 + t);
    };
    auto request = [&]() {   // rows past the last one repeat its factors, have no record and are dropped
        const long long row0 = (long long)g * RG;
#pragma unroll
        for (int t = 0; t < RG; ++t) f[t].load(S.F, row0 + t < S.rows ? row0 + t : S.rows - 1, lp, lane);
        if (MODE != PASS_INIT) {
            const float *__restrict__ vals = S.vals + base;
#pragma unroll
            for (int t = 0; t < RG; ++t) {
                RecordCursor<RR> cursor(walk[t], R);
#pragma unroll
                for (int v = 0; v < V; ++v) {
                    tv[t][v] = vals[(unsigned)(lane + 64 * v)];
                    pv[t][v] = perm_in[cursor.place(64 * v, lane + 64 * v, zero_slot)];
                }
                vals += record_total<RR>(walk[t], R);
            }
        }
        const long long mine = row0 + my < S.rows ? row0 + my : S.rows - 1;
        const int *rec = S.meta + mine * S.meta_stride;
        marg = __int_as_float(rec[2]);
        log_marg = MODE == PASS_INIT ? (double)S.log_out[mine] : __hiloint2double(rec[5], rec[4]);
        if (MODE != PASS_QUERY) pos = rec[6 + 2 * R + (sub < R ? sub : 0)];
        lin = MODE == PASS_QUERY ? S.lin_out[mine] : 0.0;
    };
    // (unconditional, so that the loads in flight can be counted: a wavefront without rows requests the last group)
    const bool busy = g < groups;
    if (!busy) g = groups - 1;
    load_walks();
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
        const int next = g + nwaves;
        double out;
        if (MODE == PASS_INIT) {
            out = exists ? exp(log_marg - m_self) : 0.0;
            if (exists && log_marg > maxlog && log_marg < INFINITY) maxlog = log_marg;
        } else {
            double acc[NV];
#pragma unroll
            for (int t = 0; t < NV; ++t) acc[t] = 0.0;
            const float *__restrict__ vals = S.vals + base;
#pragma unroll
            for (int t = 0; t < RG; ++t) {
                const int total = record_total<RR>(walk[t], R);
#pragma unroll
                for (int v = 0; v < V; ++v)
                    acc[t] = fma((double)(lane + 64 * v < total ? tv[t][v] : 0.f), (double)pv[t][v], acc[t]);
                RecordCursor<RR> cursor(walk[t], R);
                for (int e0 = 64 * V; e0 < total; e0 += 64 * TRIP) {   // all loads of a trip before the first use
                    float tt[TRIP], pp[TRIP];
#pragma unroll
                    for (int k = 0; k < TRIP; ++k) {
                        const int c = e0 + 64 * k, e = c + lane;
                        tt[k] = vals[(unsigned)e];
                        pp[k] = perm_in[cursor.place(c, e, zero_slot)];
                        if (e >= total) tt[k] = 0.f;
                    }
#pragma unroll
                    for (int k = 0; k < TRIP; ++k) acc[t] = fma((double)tt[k], (double)pp[k], acc[t]);
                }
                vals += total;
                acc[t] *= PERM_UNSCALE;
            }
            if (next < groups) {   // the next group's records are looked up while this one's factors are worked on
                const int now = g;
                g = next;
                load_walks();
                g = now;
            }
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
            const float outf = (float)(out * PERM_SCALE);
            if (exists) {
                if (sub == 0) {
                    S.lin_out[mine] = out;
                    if (outf == INFINITY) ++range;
                }
                if (sub < R) perm_out[(long long)sub * S.rows + pos] = outf;
            }
#pragma unroll
            for (int t = 0; t < RG; ++t) {
                const double o = lane_value(out, t * GL);
#pragma unroll
                for (int k = 0; k < T; ++k) zacc[k] = fma((double)f[t].f[k], o, zacc[k]);
            }
        }
        g = next;
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
    if (range) atomicAdd(&counters[6], (unsigned long long)range);
}

template <int T, int RR, int RG, int V>
static void launch_sweep_rows(const PassSide &S, const Handle &h, int mode, const FuseArgs &F, bool fused_in, int groups,
                              double *partial, unsigned long long *cnt, hipStream_t s)
{
    const dim3 grid(groups), block(PASS_THREADS);
    const size_t lds = pass_lds_bytes(h.lp, fused_in);
    if (mode == PASS_UPDATE && fused_in)
        hipLaunchKernelGGL((pass_kernel<T, RR, RG, V, PASS_UPDATE, true>), grid, block, lds, s, S, h.R, h.lp, partial, cnt, F);
    else if (mode == PASS_UPDATE)
        hipLaunchKernelGGL((pass_kernel<T, RR, RG, 1, PASS_UPDATE, false>), grid, block, lds, s, S, h.R, h.lp, partial, cnt, F);
    else if (mode == PASS_QUERY)
        hipLaunchKernelGGL((pass_kernel<T, RR, RG == 1 ? 1 : 3, 1, PASS_QUERY, false>), grid, block, lds, s, S, h.R, h.lp, partial, cnt, F);
    else
        hipLaunchKernelGGL((pass_kernel<T, 1, 3, 1, PASS_INIT, false>), grid, block, lds, s, S, h.R, h.lp, partial, cnt, F);
}

// Entries of a record requested with its row, in wavefronts of them: two, but one for short records five rows at a time
// (20 000 rows of 256 factor entries, 45 stored values on average: 13.3 us per sweep against 13.6 with two; 18 757 rows
// of 128, 98 stored values: 12.8 against 11.1), and three for longer ones of up to 128 factor entries, whose rows leave the
// registers for it.  That is most where the third holds the rest of a record (two / three, as shares: 40 000 rows of 129 values in
// three rounds 0.82, 16 000 of 148 0.87, 60 000 of 180 in two 0.87, 28 000 of 118 in one 0.92), little for longer ones (10 000 of 451 11.95 / 11.78 us, 745
// 14.14 / 13.85) and up to 3 % slower for some of 300 to 400 (21 000 of 385 in one round 15.3 / 15.8); one row at a time 4000 of 334 8.25 / 8.03,
// but 3000 of 248 7.29 / 7.40; four are no faster, six spill.
// (An entry's order in its lane's sum does not depend on that: both give the same bits.)
template <int T, int RR>
static void launch_sweep_rounds(const PassSide &S, const Handle &h, int mode, const FuseArgs &F, bool fused_in, int groups,
                                double *partial, unsigned long long *cnt, hipStream_t s)
{
    const int rows = rows_at_a_time(h, S.rows);
    if constexpr (T <= 2)
        if (h.nnz_stored > (rows == 1 ? 256 : 64) * S.rows) {
            switch (rows) {
                case 1: launch_sweep_rows<T, RR, 1, 3>(S, h, mode, F, fused_in, groups, partial, cnt, s); break;
                case 2: launch_sweep_rows<T, RR, 2, 3>(S, h, mode, F, fused_in, groups, partial, cnt, s); break;
                case 3: launch_sweep_rows<T, RR, 3, 3>(S, h, mode, F, fused_in, groups, partial, cnt, s); break;
                default: launch_sweep_rows<T, RR, 5, 3>(S, h, mode, F, fused_in, groups, partial, cnt, s);
            }
            return;
        }
    switch (rows) {
        case 1: launch_sweep_rows<T, RR, 1, 2>(S, h, mode, F, fused_in, groups, partial, cnt, s); break;
        case 2: launch_sweep_rows<T, RR, 2, 2>(S, h, mode, F, fused_in, groups, partial, cnt, s); break;
        case 3: launch_sweep_rows<T, RR, 3, 2>(S, h, mode, F, fused_in, groups, partial, cnt, s); break;
        default:
            if (h.nnz_stored <= 64 * S.rows)
                launch_sweep_rows<T, RR, 5, 1>(S, h, mode, F, fused_in, groups, partial, cnt, s);
            else if constexpr (T > 2)
                launch_sweep_rows<T, RR, 5, 2>(S, h, mode, F, fused_in, groups, partial, cnt, s);
    }
}

// The loads are unrolled over exactly the hash rounds there are, up to EXACT_ROUNDS.
template <int T>
static void launch_sweep_columns(const PassSide &S, const Handle &h, int mode, const FuseArgs &F, bool fused_in, int groups,
                                 double *partial, unsigned long long *cnt, hipStream_t s)
{
    switch (h.R) {
        case 1: launch_sweep_rounds<T, 1>(S, h, mode, F, fused_in, groups, partial, cnt, s); break;
        case 2: launch_sweep_rounds<T, 2>(S, h, mode, F, fused_in, groups, partial, cnt, s); break;
        case 3: launch_sweep_rounds<T, 3>(S, h, mode, F, fused_in, groups, partial, cnt, s); break;
        case 4: launch_sweep_rounds<T, 4>(S, h, mode, F, fused_in, groups, partial, cnt, s); break;
        default: launch_sweep_rounds<T, ANY_ROUNDS>(S, h, mode, F, fused_in, groups, partial, cnt, s);
    }
}

}  // namespace lcn
