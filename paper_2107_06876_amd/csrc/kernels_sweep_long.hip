// The half-iteration with a sparse part (see sweep.h) for factor rows of more than 256 entries.
#include "iter_common.h"

namespace lcn {

// Factor rows of more than 256 entries: a row per wavefront at a time, the next row's factor entries and first record
// entries requested before the current row is reduced.  The loop's body stands there twice, the two sets of registers in
// exchanged roles: where the requested set is copied to the current one at a row's end, the compiler waits for it there.
// 200 000 rows of 512 entries, 19 stored values: 101.4 us per sweep, 111 with the copy, 105 with the copy and a round's
// segment after the other instead of the record walked flat; two rows at a time leave no registers for the next ones
// (109, four rows spill).  What bounds it is memory: the factor rows alone, 410 MB, take 82 us at 5 TB/s.
// The copies of the scalings, the masked lanes and the zero slot are as in pass_kernel.
template <int T, int RR, int V, int MODE, bool FUSED>
__global__ __launch_bounds__(PASS_THREADS) void long_pass_kernel(PassSide S, int R, int lp, double *partial,
                                                                 unsigned long long *counters, FuseArgs Fz)
{
    constexpr int TRIP = LONG_TRIP;
    static_assert(64 * TRIP <= VALUE_SLACK && 64 * V <= VALUE_SLACK, "read past the last record");
    extern __shared__ double zsh[];  // [PASS_WAVES / 2][lp + 3], then [lp + 2] and the reduction's scratch if FUSED
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const long long nwaves = (long long)gridDim.x * PASS_WAVES;
    // Rows are dealt out from the last workgroup down: the reducing workgroups of a fused
    // sweep (the first few) start late, so they get the row slots that may hold one row less.
    // The dealing is the same with and without fusion, so both give the same bits.
    const long long gw = (long long)(gridDim.x - 1 - blockIdx.x) * PASS_WAVES + wave;
    const int stride = lp + 3;
    // exponents taken out of this side's vector (m_self) and of the input vectors (m_in)
    // (a query reads the exponent its vector was stored with, kept beside the accumulator it produced)
    if (MODE == PASS_UPDATE) mark_pending(Fz, lp);
    if (FUSED) reduce_publish(Fz, lp, zsh + (size_t)(PASS_WAVES / 2) * stride + lp + 2);
    const double m_self = MODE == PASS_QUERY ? S.acc_out[lp] : *S.shift_self;
    double m_in = 0.0, e_out = 1.0;
    double maxlog = -INFINITY;

    double yreg[T], zacc[T];
#pragma unroll
    for (int t = 0; t < T; ++t) {
        yreg[t] = 0.0;
        zacc[t] = 0.0;
    }
    if (!FUSED) {
        m_in = MODE != PASS_INIT ? S.acc_in[lp] : 0.0;
        e_out = MODE == PASS_UPDATE ? exp(-m_in - m_self) : (MODE == PASS_QUERY ? exp(m_in + m_self) : 1.0);
#pragma unroll
        for (int t = 0; t < T; ++t)
            yreg[t] = MODE != PASS_INIT ? S.acc_in[FRow<T>::kidx(t, lane)] : 0.0;
    }
    double q0 = 0.0, q1 = 0.0;
    unsigned long long nonpos = 0, range = 0;

    // Three-stage software pipeline over the rows a wave owns: metadata is read
    // two rows ahead, the factor row and the first 64 V entries of its record
    // one row ahead, and the current row is reduced while those loads are in flight.
    struct RowData {
        FRow<T> f;
        float tv[V], vv[V];
    };
    const float *__restrict__ perm_in = reinterpret_cast<const float *>(S.perm_in);
    float *__restrict__ perm_out = reinterpret_cast<float *>(S.perm_out);
    const unsigned zero_slot = (unsigned)(R * S.rows_in);
    auto issue = [&](RowData &D, const RowMeta<RR> &M, long long r) {
        D.f.load(S.F, r, lp, lane);
        if (MODE != PASS_INIT) {
            const float *__restrict__ vals = S.vals + M.base;
            RecordCursor<RR> cursor(M.walk, R);
#pragma unroll
            for (int v = 0; v < V; ++v) {
                D.tv[v] = vals[64 * v + lane];
                D.vv[v] = perm_in[cursor.place(64 * v, 64 * v + lane, zero_slot)];
            }
        }
    };
    RowData cur{}, nxt{};
    RowMeta<RR> mc{}, mn{}, mn2{};
    const int Rm = MODE == PASS_INIT ? 0 : R;
    long long row = gw, next = gw + nwaves, next2 = gw + 2 * nwaves;
    if (row < S.rows) {
        load_meta<RR, MODE>(mc, S, Rm, row, lane);
        if (MODE == PASS_INIT && lane < R) mc.pos = S.meta[row * S.meta_stride + 6 + 2 * R + lane];
        issue(cur, mc, row);
    }
    if (next < S.rows) {
        load_meta<RR, MODE>(mn, S, Rm, next, lane);
        if (MODE == PASS_INIT && lane < R) mn.pos = S.meta[next * S.meta_stride + 6 + 2 * R + lane];
    }
    if (FUSED) {
        double *ysh = zsh + (size_t)(PASS_WAVES / 2) * stride;
        if (wave == 0) fused_fetch(Fz, S.acc_in, lp, ysh);
        __syncthreads();
        m_in = ysh[lp];
        e_out = ysh[lp + 1];
#pragma unroll
        for (int t = 0; t < T; ++t) yreg[t] = ysh[FRow<T>::kidx(t, lane)];
    }
    // one row: `C` holds the row's data, `N` receives the next row's
    auto step = [&](RowData &C, RowData &N) {
        auto look_ahead = [&]() {
            if (next2 < S.rows) {
                load_meta<RR, MODE>(mn2, S, Rm, next2, lane);
                if (MODE == PASS_INIT && lane < R) mn2.pos = S.meta[next2 * S.meta_stride + 6 + 2 * R + lane];
            }
        };
        // (the words of more than EXACT_ROUNDS rounds come as a vector load, which is there no sooner than what was
        // requested before it)
        if (RR == ANY_ROUNDS) look_ahead();
        if (next < S.rows) issue(N, mn, next);
        if (RR != ANY_ROUNDS) look_ahead();
        double out;
        if (MODE == PASS_INIT) {
            const double lo = (double)S.log_out[row];
            out = exp(lo - m_self);
            if (lo > maxlog && lo < INFINITY) maxlog = lo;
        } else {
            double acc = 0.0;
            const int total = record_total<RR>(mc.walk, R);
#pragma unroll
            for (int v = 0; v < V; ++v)
                acc = fma((double)(64 * v + lane < total ? C.tv[v] : 0.f), (double)C.vv[v], acc);
            RecordCursor<RR> cursor(mc.walk, R);
            for (int e0 = 64 * V; e0 < total; e0 += 64 * TRIP) {   // all loads of a trip before the first use
                const float *__restrict__ vals = S.vals + mc.base;
                float tt[TRIP], pp[TRIP];
#pragma unroll
                for (int k = 0; k < TRIP; ++k) {
                    const int c = e0 + 64 * k, e = c + lane;
                    tt[k] = vals[(unsigned)e];
                    pp[k] = perm_in[cursor.place(c, e, zero_slot)];
                    if (e >= total) tt[k] = 0.f;
                }
#pragma unroll
                for (int k = 0; k < TRIP; ++k) acc = fma((double)tt[k], (double)pp[k], acc);
            }
            acc *= PERM_UNSCALE;
#pragma unroll
            for (int t = 0; t < T; ++t) acc = fma((double)C.f.f[t], yreg[t], acc);
            const double s = wave_sum(acc);
            const double marg = (double)mc.marg;
            if (MODE == PASS_UPDATE) {
                float lo;
                if (s > 0.0) {
                    out = marg * fast_rcp(s) * e_out;
                    const double lg = mc.log_marg - fast_log(s) - m_in;
                    lo = (float)lg;
                    maxlog = fmax(maxlog, lg);
                } else {
                    out = NAN;
                    lo = NAN;
                    ++nonpos;
                }
                if (lane == 0) S.log_out[row] = lo;
            } else {  // PASS_QUERY
                out = mc.lin;
                const double ri = out * s * e_out;
                if (lane == 0 && S.marg_out) S.marg_out[row] = (float)ri;
                if (out > 0.0) q0 += ri * (log(out) + m_self);
                q1 += fabs(ri - marg);
            }
        }
        if (MODE != PASS_QUERY) {
            if (lane == 0) S.lin_out[row] = out;
            const float outf = (float)(out * PERM_SCALE);
            if (outf == INFINITY) ++range;
            if (lane < R) perm_out[(long long)lane * S.rows + mc.pos] = outf;
#pragma unroll
            for (int t = 0; t < T; ++t) zacc[t] = fma((double)C.f.f[t], out, zacc[t]);
        }
        mc = mn;
        mn = mn2;
        row = next;
        next = next2;
        next2 += nwaves;
    };
    // the two data buffers swap roles from row to row (no register copies, which would have to wait for the loads)
    while (row < S.rows) {
        step(cur, nxt);
        if (row >= S.rows) break;
        step(nxt, cur);
    }

    group_partials<T>(zacc, q0, q1, maxlog, lp, zsh, partial);
    if (lane == 0 && (nonpos | range)) {
        if (nonpos) atomicAdd(&counters[0], nonpos);
        if (range) atomicAdd(&counters[6], range);
    }
}

template <int T, int RR, int V>
static void launch_long_mode(const PassSide &S, const Handle &h, int mode, const FuseArgs &F, bool fused_in, int groups,
                               double *partial, unsigned long long *cnt, hipStream_t s)
{
    const dim3 grid(groups), block(PASS_THREADS);
    const size_t lds = pass_lds_bytes(h.lp, fused_in);
    if (mode == PASS_UPDATE && fused_in)
        hipLaunchKernelGGL((long_pass_kernel<T, RR, V, PASS_UPDATE, true>), grid, block, lds, s, S, h.R, h.lp, partial, cnt, F);
    else if (mode == PASS_UPDATE)
        hipLaunchKernelGGL((long_pass_kernel<T, RR, V, PASS_UPDATE, false>), grid, block, lds, s, S, h.R, h.lp, partial, cnt, F);
    else if (mode == PASS_QUERY)
        hipLaunchKernelGGL((long_pass_kernel<T, RR, 1, PASS_QUERY, false>), grid, block, lds, s, S, h.R, h.lp, partial, cnt, F);
    else
        hipLaunchKernelGGL((long_pass_kernel<T, 1, 1, PASS_INIT, false>), grid, block, lds, s, S, h.R, h.lp, partial, cnt, F);
}

// Entries of a record requested with its row: a wavefront of them where records are short (200 000 rows of 512 factor
// entries and 19 stored values on average: 101.8 us per sweep, 103.2 with two, 104.9 with three; 100 000 rows of 36:
// 58.3, 59.1, 59.8), else three (200 000 rows of 120: 133.3 with one, 129.5 with two, 129.0 with three).  The bits are the
// same, as in sweep.h.
template <int T, int RR>
static void launch_long_rounds(const PassSide &S, const Handle &h, int mode, const FuseArgs &F, bool fused_in, int groups,
                               double *partial, unsigned long long *cnt, hipStream_t s)
{
    if (h.nnz_stored <= 64 * S.rows)
        launch_long_mode<T, RR, 1>(S, h, mode, F, fused_in, groups, partial, cnt, s);
    else
        launch_long_mode<T, RR, 3>(S, h, mode, F, fused_in, groups, partial, cnt, s);
}

template <int T>
static void launch_long_columns(const PassSide &S, const Handle &h, int mode, const FuseArgs &F, bool fused_in, int groups,
                                double *partial, unsigned long long *cnt, hipStream_t s)
{
    switch (h.R) {
        case 1: launch_long_rounds<T, 1>(S, h, mode, F, fused_in, groups, partial, cnt, s); break;
        case 2: launch_long_rounds<T, 2>(S, h, mode, F, fused_in, groups, partial, cnt, s); break;
        case 3: launch_long_rounds<T, 3>(S, h, mode, F, fused_in, groups, partial, cnt, s); break;
        case 4: launch_long_rounds<T, 4>(S, h, mode, F, fused_in, groups, partial, cnt, s); break;
        default: launch_long_rounds<T, ANY_ROUNDS>(S, h, mode, F, fused_in, groups, partial, cnt, s);
    }
}

hipError_t launch_long_sweep(const PassSide &S, const Handle &h, int mode, const FuseArgs &F, bool fused_in, int groups,
                             double *partial, unsigned long long *cnt, hipStream_t s)
{
    switch (h.lp / 64) {
        case 5: launch_long_columns<5>(S, h, mode, F, fused_in, groups, partial, cnt, s); break;
        case 6: launch_long_columns<6>(S, h, mode, F, fused_in, groups, partial, cnt, s); break;
        case 7: launch_long_columns<7>(S, h, mode, F, fused_in, groups, partial, cnt, s); break;
        default: launch_long_columns<8>(S, h, mode, F, fused_in, groups, partial, cnt, s);
    }
    return hipGetLastError();
}

}  // namespace lcn
