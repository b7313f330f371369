"""Which kernel a sweep or a query of a sparse kernel takes, without a GPU: log_walk.h is plain C++, so a small host program
asks it for the sizes on both sides of each of its lines."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include "log_walk.h"

int main(int argc, char **argv)   // rounds, rows, stored values, query
{
    static const char *names[] = {"FLAT_16x2", "FLAT_32x4", "FLAT_64x4", "ROUNDS_16x2", "ROUNDS_16x4", "ROUNDS_32x2", "ROUNDS_32x4"};
    for (int i = 1; i + 3 < argc; i += 4)
        puts(names[lcn::log_walk(atoi(argv[i]), atoll(argv[i + 1]), atoll(argv[i + 2]), atoi(argv[i + 3]))]);
    return 0;
}
"""

# rounds, rows, values of a row's piece of a round -> sweep, query
SIZES = [
    # short pieces in several rounds in one trip, whatever the number of rows
    (3, 3000, 4.2, "FLAT_16x2", "FLAT_16x2"), (4, 3000, 10, "FLAT_16x2", "FLAT_16x2"), (3, 20000, 7, "FLAT_16x2", "FLAT_16x2"),
    (4, 20000, 10, "FLAT_16x2", "FLAT_16x2"), (4, 40000, 10, "FLAT_16x2", "FLAT_16x2"), (2, 3000, 7, "FLAT_16x2", "FLAT_16x2"),
    (2, 30000, 25, "FLAT_16x2", "FLAT_16x2"), (4, 3000, 15, "FLAT_32x4", "FLAT_32x4"),
    # long ones of many rows too
    (3, 12500, 190, "FLAT_32x4", "ROUNDS_16x4"), (4, 28000, 160, "FLAT_32x4", "ROUNDS_16x4"), (4, 40000, 210, "FLAT_32x4", "ROUNDS_16x4"),
    (3, 20000, 163, "FLAT_32x4", "ROUNDS_16x4"), (2, 20000, 520, "FLAT_32x4", "FLAT_32x4"), (3, 7500, 140, "FLAT_32x4", "ROUNDS_32x4"),
    # the records' length up to which sixteen lanes share a row
    (2, 4999, 20, "FLAT_16x2", "FLAT_16x2"), (2, 4999, 20.5, "FLAT_32x4", "FLAT_32x4"), (2, 5000, 32, "FLAT_16x2", "FLAT_16x2"),
    (2, 9999, 32.5, "FLAT_32x4", "FLAT_32x4"), (3, 10000, 60, "FLAT_16x2", "FLAT_16x2"), (3, 11999, 61, "FLAT_32x4", "FLAT_32x4"),
    (3, 12000, 60, "FLAT_16x2", "ROUNDS_16x4"),
    # few rows of long pieces
    (2, 7999, 159, "FLAT_32x4", "ROUNDS_32x4"), (2, 7999, 160, "ROUNDS_32x4", "ROUNDS_32x4"), (2, 8000, 199, "FLAT_32x4", "ROUNDS_32x4"),
    (2, 8000, 200, "ROUNDS_32x2", "ROUNDS_32x4"), (2, 11999, 300, "ROUNDS_32x2", "ROUNDS_32x4"), (2, 12000, 300, "ROUNDS_32x4", "FLAT_32x4"),
    (2, 17999, 299, "ROUNDS_32x4", "ROUNDS_16x4"), (2, 18000, 299, "FLAT_32x4", "ROUNDS_16x4"), (2, 3000, 90, "FLAT_32x4", "ROUNDS_32x4"),
    # one round
    (1, 20000, 28, "ROUNDS_16x2", "ROUNDS_16x2"), (1, 12000, 139, "ROUNDS_16x4", "ROUNDS_16x4"), (1, 12000, 140, "ROUNDS_32x4", "ROUNDS_32x4"),
    (1, 11999, 400, "ROUNDS_32x2", "ROUNDS_32x4"), (1, 8000, 89, "ROUNDS_32x2", "ROUNDS_32x2"), (1, 7999, 90, "ROUNDS_32x4", "ROUNDS_32x4"),
    # a wavefront per row
    (4, 5000, 250, "ROUNDS_32x4", "ROUNDS_32x4"), (4, 5000, 250.5, "FLAT_64x4", "FLAT_64x4"), (5, 5000, 16, "FLAT_32x4", "FLAT_32x4"),
    (5, 5000, 16.5, "FLAT_64x4", "FLAT_64x4"), (8, 5000, 6, "FLAT_16x2", "FLAT_16x2"),
]


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not found")
def test_walk_by_rounds_rows_and_length(tmp_path):
    src, exe = tmp_path / "walk.cpp", tmp_path / "walk"
    src.write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-Wall", "-I" + os.path.join(ROOT, "paper_2107_06876_amd", "csrc"),
                           "-o", str(exe), str(src)])
    args, want = [], []
    for rounds, rows, piece, sweep, query in SIZES:
        for q, name in enumerate((sweep, query)):
            args += [rounds, rows, round(piece * rounds * rows), q]
            want.append((rounds, rows, piece, q, name))
    got = subprocess.check_output([str(exe)] + [str(a) for a in args], text=True).split()
    assert [w[:4] + (g,) for w, g in zip(want, got)] == want and len(got) == len(want)
