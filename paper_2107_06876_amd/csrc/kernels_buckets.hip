// Sparse Sinkhorn with one hash round (and a small dense kernel, which is a single bucket): a whole run in one launch.
//
// With one round the pattern is one block of X rows times Y columns per bucket and nothing connects the blocks, so a
// workgroup takes a bucket through all iterations with the block's values, scalings and marginals in LDS: no launch, no trip
// to memory and no other workgroup between two half-iterations.  The arithmetic is that of logpass_kernel: a row's
// log-sum-exp with its previous value as the shift, exp in single precision, sums in double, a second walk with running
// maxima where that sum leaves single precision's range.
//
// What bounds it is the chain of one half-iteration: a few entries per lane, the sum over the lanes of a row, a
// logarithm, a barrier.  Eight lanes share a row, so that a block of 32 x 32 is one step of 256 threads.  Rows of the
// tile are an odd multiple of eight floats apart: eight rows times eight columns then lie in 64 different banks, whichever of the
// two runs along the lanes.
// us per half-iteration, a launch per sweep / so: 10 000 x 10 000 in 500 buckets 3.6 / 0.64, 30 000 x 30 000 in 1200 5.1 / 1.2,
// 3000 x 3000 in 32 3.6 / 1.5, a block of 32 x 32 3.3 / 0.52, of 100 x 100 3.2 / 1.4; the largest ones that fit, 192 x 192 and
// 320 x 110, 3.5 / 2.9 and 3.5 / 3.2. (With entries past a row's end masked instead of padded: 1.97 instead of 1.4 at 30 000.)
#include <mutex>
#include <type_traits>

#include "iter_common.h"

namespace lcn {

constexpr int BK_LANES = 8;      // lanes per row
constexpr int BK_AHEAD = 4;      // entries of a row that a lane requests together

__device__ inline double eight_sum(double v)   // every lane of the eight gets the result
{
    v = dpp_add<0xB1, 0xF>(v);
    v = dpp_add<0x4E, 0xF>(v);
    return dpp_add<0x141, 0xF>(v);
}

__device__ inline double eight_max(double v)
{
    v = dpp_max<0xB1, 0xF>(v);
    v = dpp_max<0x4E, 0xF>(v);
    return dpp_max<0x141, 0xF>(v);
}

// One half-iteration: `count` rows of `len` entries, entry c of row r at tile[r * row_step + c * entry_step].
// self: the rows' log scalings (replaced), mass: logs of their marginals, other: the entries' log scalings.
template <int THREADS>
__device__ inline void bucket_half(const float *tile, int count, int len, int row_step, int entry_step, double *self,
                                   const double *mass, const double *other, unsigned &empty)
{
    const int sub = threadIdx.x % BK_LANES;
    for (int r = threadIdx.x / BK_LANES; r < count; r += THREADS / BK_LANES) {
        const float *row = tile + r * row_step;
        const double log_marg = mass[r], prev = self[r], shift = log_marg - prev;
        double lse = 0.0;
        bool done = false;
        if (shift > -INFINITY && shift < INFINITY) {   // the same in every lane of the row
            double acc = 0.0;
            const float *at = row + sub * entry_step;
            const double *with = other + sub;
            auto piece = [&](auto entries) {   // so many entries of every lane
                constexpr int U = decltype(entries)::value;
                float k[U];
                double p[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    k[u] = at[u * BK_LANES * entry_step];
                    p[u] = with[u * BK_LANES];
                }
#pragma unroll
                for (int u = 0; u < U; ++u) acc += (double)__expf(k[u] + (float)(p[u] - shift));
                at += U * BK_LANES * entry_step;
                with += U * BK_LANES;
            };
            int left = (len + BK_LANES - 1) / BK_LANES;
            for (; left >= BK_AHEAD; left -= BK_AHEAD) piece(std::integral_constant<int, BK_AHEAD>{});
            if (left & 2) piece(std::integral_constant<int, 2>{});
            if (left & 1) piece(std::integral_constant<int, 1>{});
            const double tot = eight_sum(acc);
            if (tot > 1e-30 && tot < 1e30) {
                lse = shift + fast_log(tot);
                done = true;
            }
        }
        if (!done) {
            double mx = -INFINITY, sm = 0.0;
            for (int c = sub; c < len; c += BK_LANES) lse_step((double)row[c * entry_step] + other[c], mx, sm);
            const double M = eight_max(mx);
            const double sum = eight_sum(mx > -INFINITY ? sm * exp(mx - M) : 0.0);
            lse = sum > 0.0 ? M + log(sum) : -INFINITY;
        }
        if (sub == 0) {
            if (!(lse > -INFINITY)) ++empty;   // no kernel entry reaches this point: it carries no mass
            self[r] = lse > -INFINITY ? log_marg - lse : -INFINITY;
        }
    }
    __syncthreads();
}

template <int THREADS>
__global__ __launch_bounds__(THREADS) void bucket_run_kernel(PassSide X, PassSide Y, SortBuffers B, int iters,
                                                             unsigned long long *counters)
{
    extern __shared__ double bucket_lds[];   // log u, log v, log a, log b of the block, then its values
    const int *off_x = B.off, *off_y = B.off + B.b + 1;
    const int x0 = off_x[blockIdx.x], y0 = off_y[blockIdx.x];
    const int nx = off_x[blockIdx.x + 1] - x0, ny = off_y[blockIdx.x + 1] - y0;
    const int *rows = B.perm + x0, *columns = B.perm + B.n + y0;
    const int px = bucket_padded(nx), py = bucket_padded(ny), step = bucket_tile_step(ny);
    double *u = bucket_lds, *v = u + px, *a = v + py, *b = a + px;
    float *tile = (float *)(b + py);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // entries past the end, up to a multiple of eight, are read with the others: kernel values of zero
    for (int i = threadIdx.x; i < px; i += THREADS) {
        if (i >= nx) {
            u[i] = 0.0;
            continue;
        }
        const int row = rows[i], *rec = X.meta + (long long)row * X.meta_stride;
        u[i] = X.lin_out[row];
        a[i] = __hiloint2double(rec[5], rec[4]);
    }
    for (int j = threadIdx.x; j < py; j += THREADS) {
        if (j >= ny) {
            v[j] = 0.0;
            continue;
        }
        const int column = columns[j], *rec = Y.meta + (long long)column * Y.meta_stride;
        v[j] = Y.lin_out[column];
        b[j] = __hiloint2double(rec[5], rec[4]);
    }
    for (int i = wave; i < px; i += THREADS / 64) {   // a row's record is its ny values in the order of the columns
        const float *values = i < nx ? X.vals + record_base(X, rows[i]) : nullptr;
        for (int j = lane; j < py; j += 64) tile[i * step + j] = i < nx && j < ny ? values[j] : -INFINITY;
    }
    __syncthreads();
    unsigned empty_rows = 0, empty_columns = 0;
    for (int it = 0; it < iters; ++it) {
        bucket_half<THREADS>(tile, nx, ny, step, 1, u, a, v, empty_rows);
        bucket_half<THREADS>(tile, ny, nx, 1, step, v, b, u, empty_columns);
    }
    for (int i = threadIdx.x; i < nx; i += THREADS) {
        const int row = rows[i];
        X.log_out[row] = (float)u[i];
        X.lin_out[row] = u[i];
        X.perm_out[x0 + i] = u[i];
    }
    for (int j = threadIdx.x; j < ny; j += THREADS) {
        const int column = columns[j];
        Y.log_out[column] = (float)v[j];
        Y.lin_out[column] = v[j];
        Y.perm_out[y0 + j] = v[j];
    }
    if (empty_rows) atomicAdd(&counters[1], (unsigned long long)empty_rows);
    if (empty_columns) atomicAdd(&counters[2], (unsigned long long)empty_columns);
}

// More than 64 KB of dynamic LDS has to be allowed per kernel and device before the first such launch.
template <int THREADS>
static hipError_t allow_bucket_lds()
{
    static std::mutex mu;
    static bool allowed[64] = {};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const bool known = dev >= 0 && dev < 64;
    std::lock_guard<std::mutex> lock(mu);
    if (known && allowed[dev]) return hipSuccess;
    e = hipFuncSetAttribute(reinterpret_cast<const void *>(&bucket_run_kernel<THREADS>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)BUCKET_LDS_BYTES);
    if (e == hipSuccess && known) allowed[dev] = true;
    return e;
}

static BucketRun bucket_run_of(const Handle &h)
{
    BucketRun r{};
    r.block_bytes = h.block_bytes;
    r.block_side = h.block_side;
    r.b = h.b;
    r.nnz = h.nnz_stored;
    r.rows = h.n > h.m ? h.n : h.m;
    r.cus = h.cus > 0 ? h.cus : 256;
    return r;
}

bool bucket_run_taken(const Handle &h) { return h.log_domain && h.R == 1 && bucket_run_pays(bucket_run_of(h)); }

template <int THREADS>
static hipError_t launch_bucket_threads(const PassSide &X, const PassSide &Y, const Handle &h, const BucketRun &r, int iters, hipStream_t s)
{
    if (r.block_bytes > 64 * 1024) {
        const hipError_t e = allow_bucket_lds<THREADS>();
        if (e != hipSuccess) return e;
    }
    const int most = bucket_launch_iterations(r);
    while (iters > 0) {
        const int some = iters < most ? iters : most;
        hipLaunchKernelGGL(bucket_run_kernel<THREADS>, dim3(h.b), dim3(THREADS), (size_t)r.block_bytes, s, X, Y, h.sort, some,
                           h.counters);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        iters -= some;
    }
    return hipSuccess;
}

hipError_t launch_bucket_run(const PassSide &X, const PassSide &Y, const Handle &h, int iters, hipStream_t s)
{
    const BucketRun r = bucket_run_of(h);
    switch (bucket_threads(r)) {
        case 256: return launch_bucket_threads<256>(X, Y, h, r, iters, s);
        case 512: return launch_bucket_threads<512>(X, Y, h, r, iters, s);
        default: return launch_bucket_threads<1024>(X, Y, h, r, iters, s);
    }
}

}  // namespace lcn
