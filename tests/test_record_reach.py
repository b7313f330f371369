"""How far the sweeps read past the stored values, without a GPU: record_reach.h is plain C++, so a small host program walks
records of every length as the kernels do and compares the last entry touched with the room behind the values."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include "record_reach.h"

int main()
{
    // chunks requested with a row, chunks per trip: rows of up to 256 factor entries, longer ones
    const int sweeps[][2] = {{1, lcn::SWEEP_TRIP}, {2, lcn::SWEEP_TRIP}, {3, lcn::SWEEP_TRIP}, {1, lcn::LONG_TRIP}, {3, lcn::LONG_TRIP}};
    int furthest = 0;
    for (const auto &s : sweeps)
        for (int total = 0; total <= 2000; ++total) {
            int last = -1;   // number of the last entry that some lane reads
            for (int v = 0; v < s[0]; ++v)
                for (int lane = 0; lane < 64; ++lane) last = 64 * v + lane;
            for (int e0 = 64 * s[0]; e0 < total; e0 += 64 * s[1])
                for (int k = 0; k < s[1]; ++k)
                    for (int lane = 0; lane < 64; ++lane) last = e0 + 64 * k + lane;
            const int past = last + 1 > total ? last + 1 - total : 0;
            if (past != lcn::read_past_end(total, s[0], s[1]) || last >= total + lcn::VALUE_SLACK) {
                printf("%d entries, %d + %d chunks: %d past the end, room for %d\n", total, s[0], s[1], past, lcn::VALUE_SLACK);
                return 1;
            }
            furthest = past > furthest ? past : furthest;
        }
    printf("furthest %d of %d\n", furthest, lcn::VALUE_SLACK);
    return 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not found")
def test_sweeps_stay_within_the_slack(tmp_path):
    src, exe = tmp_path / "reach.cpp", tmp_path / "reach"
    src.write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-Wall", "-I" + os.path.join(ROOT, "paper_2107_06876_amd", "csrc"),
                           "-o", str(exe), str(src)])
    res = subprocess.run([str(exe)], stdout=subprocess.PIPE, text=True)
    assert res.returncode == 0, res.stdout
