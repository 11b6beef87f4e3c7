"""The lines at which calls change from one form to another, both sides of each, asked of the built library's own rules (no GPU)."""
import os
import subprocess

import pytest

from paper_2604_17198_amd import binding as nb
from paper_2604_17198_amd import build

UNITS = 256


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    """The values of C++ expressions over the rules of kernels.hpp."""
    if not os.path.exists(build.LIB):
        pytest.fail(f"{build.LIB} not built; run `python -m paper_2604_17198_amd.build`")
    where = tmp_path_factory.mktemp("rules")

    def values(expressions):
        source, program = where / "rules.hip", where / "rules"
        lines = "\n".join(f'    std::printf("%lld\\n", (long long)({e}));' for e in expressions)
        source.write_text('#include <cstdio>\n#include "common.hpp"\n#include "kernels.hpp"\nusing namespace nacho;\n'
                          f"int main()\n{{\n{lines}\n}}\n")
        subprocess.run([build._hipcc(), "-O0", "-std=c++17", "--offload-host-only", "-I", os.path.join(build.ROOT, "include"),
                        "-I", build.CSRC, str(source), "-L", build.PKG, "-l:libnacho.so", f"-Wl,-rpath,{build.PKG}",
                        "-o", str(program)], check=True, capture_output=True, text=True)
        out = subprocess.run([str(program)], check=True, capture_output=True, text=True, timeout=60).stdout
        return [int(v) for v in out.split()]

    return values


def _ahead(fmt, dtype, k, total, rows=4000, cols=4000, depth=60):
    return f"merge_fields({fmt}, {dtype}, {k}, {rows}, {cols}, {depth}, {total}, {UNITS}).touch"


def test_sums_that_ask_for_their_values_ahead(ask):
    """Two and three coordinate lists past what short partitions hold (five sixths of a round of them), whatever their keys, three up
    to 14M entries; two tensors of floats from 3.2M on, two and three of doubles as long as a round of long partitions holds them."""
    short, long = UNITS * 4 * 5 * (1472 - nb.MAX_OPERANDS) // 6, UNITS * 4 * (5040 - nb.MAX_OPERANDS)
    cases = []
    for dtype in (nb.F32, nb.F64):
        for k in (2, 3, 4, 8):
            cases += [(_ahead("SPADD_COO", dtype, k, short), 0), (_ahead("SPADD_COO", dtype, k, short + 1), int(k <= 3)),
                      (_ahead("SPADD_COO", dtype, k, short, 2**31 - 1, 2**31 - 1), 0),
                      (_ahead("SPADD_COO", dtype, k, short + 1, 2**31 - 1, 2**31 - 1), int(k <= 3)),
                      (_ahead("SPADD_COO", dtype, k, 14_000_000), int(k <= 3)), (_ahead("SPADD_COO", dtype, k, 14_000_001), int(k == 2)),
                      (_ahead("SPADD_CSF3", dtype, k, 3_199_999, 60, 60), 0),
                      (_ahead("SPADD_CSF3", dtype, k, 3_200_000, 60, 60), int(k == 2 if dtype == nb.F32 else k <= 3)),
                      (_ahead("SPADD_CSF3", dtype, k, long, 60, 60), int(k == 2 if dtype == nb.F32 else k <= 3)),
                      (_ahead("SPADD_CSF3", dtype, k, long + 1, 60, 60), int(k == 2 and dtype == nb.F32))]
            cases += [(_ahead(f"SPADD_{fmt}", dtype, k, 10_000_000), 0) for fmt in ("VECTOR", "CSR", "DCSR")]
    assert ask([e for e, _ in cases]) == [want for _, want in cases]


def _whole(dtype, nnz, n_rows, x_bytes):
    grain = f"spmv_grain({dtype}, {nnz}, {n_rows})"
    return f"spmv_whole({dtype}, {nnz}, {grain}, ({nnz} + {grain} - 1) / {grain}, {n_rows}, {x_bytes}LL)"


MB4, ANY = 4 << 20, 1 << 33


def test_spmv_without_a_partition_kernel(ask):
    """Up to 1024 partitions (short ones of floats count half) whatever x, up to 4096 of either kind while x fits an L2 (4 MiB); past
    them doubles up to 10240 with 2.5 MiB of x, floats up to 8192 long or 10240 short ones with 4 MiB and 131,072 rows.  256 rows a partition
    (two short ones) at most."""
    F, D = nb.F32, nb.F64
    cases = [
        ((D, 0, 100, 8), 0), ((D, 1, 256, 8), 1), ((D, 1, 257, 8), 0), ((D, 513, 512, 8), 1), ((D, 513, 513, 8), 0),
        ((F, 513, 256, 8), 1), ((F, 513, 257, 8), 0), ((F, 1025, 512, 8), 1), ((F, 1025, 513, 8), 0),
        # doubles: 1024, 4096, 10240 partitions of 512
        ((D, 1024 * 512, 9, ANY), 1), ((D, 1024 * 512 + 1, 9, MB4), 1), ((D, 1024 * 512 + 1, 9, MB4 + 8), 0),
        ((D, 4096 * 512, 9, MB4), 1), ((D, 4096 * 512, 9, MB4 + 8), 0), ((D, 4096 * 512, 4096 * 256, MB4), 1),
        ((D, 4096 * 512 + 1, 9, 5 << 19), 1), ((D, 4096 * 512 + 1, 9, (5 << 19) + 8), 0),
        ((D, 10240 * 512, 9, 5 << 19), 1), ((D, 10240 * 512 + 1, 9, 8), 0), ((D, 10240 * 512, 10240 * 256, 8), 1),
        # floats, short partitions (fewer than 48 a row): 2048, 4096, 10240 of 512
        ((F, 2048 * 512, 100_000, ANY), 1), ((F, 2048 * 512 + 1, 100_000, MB4), 1), ((F, 2048 * 512 + 1, 100_000, MB4 + 4), 0),
        ((F, 4096 * 512, 131_073, MB4), 1), ((F, 4096 * 512 + 1, 131_073, 4), 0), ((F, 4096 * 512 + 1, 131_072, MB4), 1),
        ((F, 4096 * 512 + 1, 131_072, MB4 + 4), 0), ((F, 10240 * 512, 131_072, MB4), 1), ((F, 10240 * 512 + 1, 131_072, MB4), 0),
        # floats, long ones (1.4M non-zeros and 48 a row): 4096, 8192 of 1024
        ((F, 1_400_000, 9, MB4), 1), ((F, 1_400_000, 9, MB4 + 4), 0), ((F, 4096 * 1024, 80_000, MB4), 1),
        ((F, 4096 * 1024 + 1, 80_000, MB4 + 4), 0), ((F, 8192 * 1024, 131_072, MB4), 1), ((F, 8192 * 1024, 131_073, MB4), 0),
        ((F, 8192 * 1024 + 1, 131_072, 4), 0),
    ]
    assert ask([_whole(*c) for c, _ in cases]) == [want for _, want in cases]
