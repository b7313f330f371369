"""When a sparse run of one hash round goes bucket by bucket, without a GPU: bucket_rule.h is plain C++, so a small host
program asks it for blocks on both sides of its lines and compares its estimate of a half-iteration with measured ones."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include "bucket_rule.h"

int main(int argc, char **argv)   // buckets, of which so many have X points x Y points, and the others; compute units
{
    for (int i = 1; i + 6 < argc; i += 7) {
        const long long b = atoll(argv[i]), many = atoll(argv[i + 1]), nx = atoll(argv[i + 2]), ny = atoll(argv[i + 3]),
                        sx = atoll(argv[i + 4]), sy = atoll(argv[i + 5]);
        lcn::BucketRun r{};
        const long long big = lcn::bucket_block_bytes((int)nx, (int)ny), small = b > many ? lcn::bucket_block_bytes((int)sx, (int)sy) : 0;
        r.block_bytes = big > small ? big : small;
        r.block_side = nx > ny ? nx : ny;
        r.b = b;
        r.nnz = many * nx * ny + (b - many) * sx * sy;
        const long long n = many * nx + (b - many) * sx, m = many * ny + (b - many) * sy;
        r.rows = n > m ? n : m;
        r.cus = atoi(argv[i + 6]);
        const bool run = lcn::bucket_run_pays(r);
        printf("%d %d %lld %d\n", run, run ? lcn::bucket_threads(r) : 0, run ? lcn::bucket_half_ns(r) : 0,
               run ? lcn::bucket_launch_iterations(r) : 0);
    }
    return 0;
}
"""

# buckets, so many of them nx x ny, the others sx x sy; threads (0: a launch per sweep); measured ns of a half-iteration (0: not)
BLOCKS = [
    # the largest blocks that fit
    (1, 1, 192, 192, 0, 0, 1024, 2900), (1, 1, 193, 193, 0, 0, 0, 0), (1, 1, 320, 100, 0, 0, 1024, 0), (1, 1, 321, 9, 0, 0, 0, 0),
    # threads
    (1, 1, 32, 32, 0, 0, 256, 0), (1, 1, 40, 40, 0, 0, 512, 690), (1, 1, 72, 72, 0, 0, 512, 0), (1, 1, 73, 73, 0, 0, 1024, 0),
    (513, 1, 73, 73, 5, 5, 512, 0), (2049, 1, 72, 72, 5, 5, 256, 0),
    # a full bucket among many small ones
    (2000, 1, 140, 140, 3, 3, 512, 3426), (2000, 1, 190, 190, 3, 3, 512, 3839), (3000, 1, 140, 140, 3, 3, 0, 0),
    (3000, 1, 140, 140, 10, 10, 512, 5353), (3500, 1, 140, 140, 6, 6, 0, 0), (3500, 40, 190, 190, 6, 6, 512, 6041),
    (4096, 10, 190, 190, 1, 1, 0, 0), (4096, 1, 140, 140, 3, 3, 0, 0), (4096, 1, 140, 140, 10, 10, 0, 0),
    (4096, 1, 110, 110, 3, 3, 512, 3431), (4000, 200, 180, 180, 5, 5, 512, 9109),
    # balanced ones
    (600, 600, 20, 20, 0, 0, 256, 0), (4096, 4096, 20, 20, 0, 0, 256, 0), (1000, 1000, 190, 190, 0, 0, 512, 0),
]


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not found")
def test_runs_bucket_by_bucket_by_block_and_number(tmp_path):
    src, exe = tmp_path / "rule.cpp", tmp_path / "rule"
    src.write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-Wall", "-I" + os.path.join(ROOT, "paper_2107_06876_amd", "csrc"),
                           "-o", str(exe), str(src)])
    args = [str(a) for block in BLOCKS for a in block[:6] + (256,)]
    got = [tuple(int(v) for v in line.split()) for line in subprocess.check_output([str(exe)] + args, text=True).splitlines()]
    assert len(got) == len(BLOCKS)
    for block, (run, threads, ns, iterations) in zip(BLOCKS, got):
        assert (run, threads) == (block[6] > 0, block[6]), block
        if run:   # the estimate is not below what was measured, and a launch takes 4 ms or a single iteration
            assert ns >= block[7], block
            assert iterations >= 1 and (iterations == 1 or 2 * iterations * ns <= 4_000_000), block
