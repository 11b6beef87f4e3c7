"""The arithmetic on rows that the kernels share with the host, compiled for the host: matrices have up to 2^31 - 1 rows, so a sum
of two rows, or of a row and a lane's offset, may lie past what 32 bits with a sign hold."""
import os
import subprocess

import pytest

from paper_2604_17198_amd import build

PROGRAM = r"""
#include <algorithm>
#include <cstdio>
#include <vector>
#include "common.hpp"
using namespace nacho;
typedef long long Wide;

static int bad = 0;
static void expect(const char *what, Wide got, Wide want)
{
    if (got != want && ++bad < 20) std::printf("%s: %lld, should be %lld\n", what, got, want);
}
CHECK
int main()
{
    check();
    std::printf("%d wrong\n", bad);
    return bad != 0;
}
"""

EDGES = r"""
static std::vector<int> edges(Wide n)          // rows near the ends and the middle of n, 0 and n among them
{
    std::vector<int> at;
    for (Wide x : {Wide(0), Wide(1), Wide(63), Wide(64), Wide(512), n / 2, n - 1025, n - 512, n - 65, n - 64, n - 63, n - 1, n})
        if (x >= 0 && x <= n) at.push_back((int)x);
    return at;
}
"""


def _run(tmp_path, check):
    source, program = tmp_path / "check.hip", tmp_path / "check"
    source.write_text(PROGRAM.replace("CHECK", EDGES + check))
    # (trapping on signed overflow: what the device does with it, the host is not to do either)
    subprocess.run([build._hipcc(), "-O1", "-std=c++17", "-ftrapv", "--offload-host-only", "-I", os.path.join(build.ROOT, "include"),
                    "-I", build.CSRC, str(source), "-o", str(program)], check=True, capture_output=True, text=True)
    done = subprocess.run([str(program)], capture_output=True, text=True, timeout=60)
    assert done.returncode == 0, done.stdout


EXTENTS = [0, 1, 64, 1000, 2**30, 2**31 - 65, 2**31 - 64, 2**31 - 2, 2**31 - 1]


@pytest.mark.parametrize("most", [512, 1024])
def test_rows_that_a_partition_spans(tmp_path, most):
    """Up to all rows of the largest matrix."""
    _run(tmp_path, """
static void check()
{
    for (Wide n : {%s})
        for (int r0 : edges(n))
            for (int r1 : edges(n))
                if (r0 <= r1)
                    expect("rows", rows_spanned(r0, r1, (int)n, %d), std::min({Wide(r1) - r0 + 1, n - r0, Wide(%d)}));
}
""" % (", ".join(f"Wide({n})" for n in EXTENTS), most, most))
