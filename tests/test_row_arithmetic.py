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
            for (int r1 : edges(n)) {
                expect("row behind", row_behind(r1, (int)n), std::min(Wide(r1) + 1, n));
                if (r0 <= r1)
                    expect("rows", rows_spanned(r0, r1, (int)n, %d), std::min({Wide(r1) - r0 + 1, n - r0, Wide(%d)}));
            }
}
""" % (", ".join(f"Wide({n})" for n in EXTENTS), most, most))


SEARCH = r"""
struct Rows {                                  // ascending stored rows, one non-zero each
    std::vector<Wide> stored;
    Wide n;
    Wide pos(Wide r) const
    {
        expect("a position of the matrix", r >= 0 && r <= n, 1);
        return std::lower_bound(stored.begin(), stored.end(), r) - stored.begin();
    }
};
template <class Body> static void matrices(Body body)
{
    for (Wide n : {EXTENTS})
        for (int from : edges(n))
            for (Wide step : {Wide(1), Wide(70), n / 5 + 1}) {
                Rows rows{{}, n};
                for (Wide r = from; r < n && rows.stored.size() < 9; r += step) rows.stored.push_back(r);
                body(rows);
            }
}
// the rows that end at or before q, by rounds of kLanes lanes
template <int kLanes> static Wide rows_before(const Rows &rows, Wide q)
{
    int lo = 0, hi = (int)rows.n, rounds = 0;
    while (lo < hi && ++rounds < 40) {
        const RowRound<kLanes> round(lo, hi);
        int n = 0;
        for (int i = 0; i < kLanes; ++i) n += round.at(i) < round.hi && rows.pos(Wide(round.at(i)) + 1) <= q;
        round.narrow(n, lo, hi);
    }
    return lo;
}
static void check()
{
    matrices([](const Rows &rows) {
        const Wide nnz = (Wide)rows.stored.size();
        for (Wide q = 0; q <= nnz; ++q) {
            const Wide want = q < nnz ? rows.stored[(size_t)q] : rows.n;
            expect("32 lanes", rows_before<32>(rows, q), want);
            expect("64 lanes", rows_before<64>(rows, q), want);
        }
        // first_row_past from any row up to the one that holds q
        for (Wide q = 0; q < nnz; ++q)
            for (int first : edges(rows.n)) {
                if (rows.pos(first) > q) continue;
                int lo = first, hi = (int)rows.n, rounds = 0;
                while (hi - lo > 1 && ++rounds < 40) {
                    int L = 0;
                    while (L < 64 && rows.pos(Wide(row_probe(lo, hi, L)) + 1) <= q) ++L;
                    expect("a lane past it", L < 64, 1);
                    if (L == 64) break;
                    const int hit = row_probe(lo, hi, L), before = row_probe(lo, hi, L > 0 ? L - 1 : 0);
                    if (L > 0) lo = before + 1;
                    hi = hit + 1;
                }
                expect("first row past", lo, std::max<Wide>(first, rows.stored[(size_t)q]));
            }
    });
}
"""


def test_rounds_of_the_searches_for_rows(tmp_path):
    """All rows of the largest matrix, and the last few of them."""
    _run(tmp_path, SEARCH.replace("EXTENTS", ", ".join(f"Wide({n})" for n in EXTENTS)))
