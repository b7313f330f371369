// When a sparse run of one hash round goes bucket by bucket (kernels_buckets.hip), in plain C++ so that it can be checked on a host.
#pragma once

namespace lcn {

// LDS of a block: two doubles per row and column, then its values, rows an odd multiple of eight floats apart; rows and columns
// up to a multiple of eight.
constexpr long long BUCKET_LDS_BYTES = 160 * 1024;
constexpr int BUCKET_MAX_SIDE = 320;
constexpr int bucket_padded(int n) { return (n + 7) / 8 * 8; }
constexpr int bucket_tile_step(int ny) { return ((ny + 7) / 8 | 1) * 8; }
constexpr long long bucket_block_bytes(int nx, int ny)
{
    return 16ll * (bucket_padded(nx) + bucket_padded(ny)) + 4ll * bucket_padded(nx) * bucket_tile_step(ny);
}

// What a run's rules go by.  LDS and threads of every workgroup follow the largest block.
struct BucketRun {
    long long block_bytes, block_side;   // most LDS a block takes, its most rows or columns
    long long b, nnz;                    // blocks, stored values
    long long rows;                      // of the larger side
    int cus;                             // compute units
};

// Threads by the largest block: as many as its rows fill in a step or two, fewer where many buckets share a compute unit,
// most of them smaller ones.  us per half-iteration with 256 / 512 / 1024 threads: a block of 40 x 40 0.99 / 0.69 / 0.69, 64 x 64
// 1.19 / 0.78 / 0.78, 192 x 192 - / 3.8 / 2.9; 1200 buckets of 25 x 25 on average 1.39 / 1.35 / 2.76, 4000 of them 3.0 / 3.6 / 8.5, 600 of
// 70 x 70 - / 2.7 / 3.2.
constexpr int bucket_threads(const BucketRun &r)
{
    if (r.block_bytes <= 6 * 1024 || (r.block_bytes <= 24 * 1024 && r.b > 8 * r.cus)) return 256;
    return r.block_bytes <= 24 * 1024 || r.b > 2 * r.cus ? 512 : 1024;
}

// Workgroups that share the chip: by LDS, and by the six wavefronts per SIMD that the kernel's 77 registers leave room for.
constexpr long long bucket_resident(const BucketRun &r)
{
    const long long by_lds = BUCKET_LDS_BYTES / r.block_bytes, by_waves = 24 * 64 / bucket_threads(r);
    return r.cus * (by_lds < by_waves ? by_lds : by_waves);
}

// Workgroups that follow one another on a compute unit, as blocks beyond bucket_resident() do.
constexpr long long bucket_turns(const BucketRun &r) { return (r.b + bucket_resident(r) - 1) / bucket_resident(r); }

// A half-iteration in ns, no less than it takes: 400 for each turn, however small its block, and the chain of as many
// blocks of the largest size as there are values for (us, so / measured: a block of 40 x 40 1.0 / 0.7, of 192 x 192 4.9 / 2.9; 4000
// buckets, one of 180 x 180, the others of 5 x 5, 10.4 / 6.2, with 200 of 180 x 180 13 / 9.1).
constexpr long long bucket_half_ns(const BucketRun &r)
{
    const long long chain = 400 + r.block_bytes / 40, blocks = 4 * r.nnz / r.block_bytes;
    return 400 * bucket_turns(r) + chain * (1 + blocks / bucket_resident(r));
}

// A block has to fit the LDS of a compute unit.  The longest side: beyond it eight lanes per row are too few (4 x 2000
// would be 250 entries per lane, two thirds of the threads without a row).
//
// With one full bucket among thousands of small ones each compute unit has one workgroup at a time, and the small ones' turns
// follow one another: a launch per sweep takes some 3.6 us, one more per 20 000 rows and 0.8 per million values.  us per
// half-iteration, a launch per sweep / bucket by bucket: 4096 buckets of 1 x 1 with ten of 190 x 190 4.0 / 6.8, of 3 x 3 with one of
// 140 x 140 4.4 / 6.6, of 10 x 10 6.1 / 7.0; 3000 of 3 x 3 4.0 / 4.9, of 10 x 10 5.5 / 5.4; 3500 of 6 x 6 with forty of 190 x 190 6.7 / 6.0; 2000 of 3 x 3
// with one of 140 x 140 3.9 / 3.4, of 190 x 190 4.4 / 3.8; one block of 110 x 110, so that two workgroups share a compute unit, with 4095 of
// 3 x 3 4.6 / 3.4.
constexpr bool bucket_run_pays(const BucketRun &r)
{
    if (r.block_bytes <= 0 || r.block_bytes > BUCKET_LDS_BYTES || r.block_side > BUCKET_MAX_SIDE) return false;
    return 400 * bucket_turns(r) <= 3600 + r.rows / 20 + r.nnz / 1250;
}

// Iterations of a launch: 4 ms of them at most, so that no launch keeps others waiting for long.  (The state passes through
// memory between launches without a loss.)
constexpr int bucket_launch_iterations(const BucketRun &r)
{
    const long long some = 4000000 / (2 * bucket_half_ns(r));
    return some > 1 ? (int)some : 1;
}

}  // namespace lcn
