"""How SpMM calls are cut and what workspace they ask for, from the host descriptors alone (no GPU)."""
import ctypes

import pytest

from paper_2604_17198_amd import binding as nb


def _operand(n_rows, n_cols, nnz):
    t = nb._Tensor()
    t.nlevels = 2
    t.lvl[0].kind, t.lvl[0].extent = nb.DENSE, n_rows
    t.lvl[1].kind, t.lvl[1].extent, t.lvl[1].count = nb.COMPRESSED, n_cols, nnz
    return ctypes.byref((nb._Tensor * 1)(t))


def _partitions(n_cols, nnz, dtype, n):
    return int(nb.lib().nacho_num_partitions(nb.OP_SPMM, _operand(n_cols, n_cols, nnz), 1, dtype, n, 0))


# (the first number of columns that sorts; non-zeros of a sorted and of an unsorted partition)
@pytest.mark.parametrize("dtype,n,n_cols,nnz,short,long", [(nb.F32, 16, 62_500, 10_000_000, 256, 512),
                                                           (nb.F32, 32, 60_938, 5_000_000, 256, 512),
                                                           (nb.F32, 64, 35_157, 3_000_000, 192, 512),
                                                           (nb.F32, 96, 23_438, 2_500_000, 128, 512),
                                                           (nb.F64, 200, 5_625, 1_000_000, 64, 256)])
def test_b_that_the_l2s_hold_is_not_sorted_for(dtype, n, n_cols, nnz, short, long):
    assert _partitions(n_cols, nnz, dtype, n) == -(-nnz // short)
    assert _partitions(n_cols - 1, nnz, dtype, n) == -(-nnz // long)


def _workspace(n_cols, nnz, dtype, n):
    size = ctypes.c_size_t(0)
    assert nb.lib().nacho_workspace_bytes(nb.OP_SPMM, _operand(n_cols, n_cols, nnz), 1, dtype, n, 0, ctypes.byref(size)) == 0
    return size.value


@pytest.mark.parametrize("dtype,n,nnz", [(nb.F32, 64, 100_000_000), (nb.F64, 200, 10_000_000), (nb.F64, 200, 30_000_000),
                                         (nb.F64, 300, 200_000_000), (nb.F32, 300, 2**31 - 1), (nb.F64, 300, 2**31 - 1)])
def test_workspace_of_sorted_calls_is_bounded(dtype, n, nnz):
    """Carries of 512 MiB, or of partitions of 512 non-zeros where those take more; 24 bytes of table, 4 of carry rows and
    8 of the sort a partition, and what is the same for all calls."""
    row = min(n, 256) * (8 if dtype == nb.F64 else 4)
    parts = _partitions(1_000_000, nnz, dtype, n)
    assert -(-nnz // 512) <= parts <= -(-nnz // 64)
    assert parts * row <= max(512 << 20, -(-nnz // 512) * row)
    assert _workspace(1_000_000, nnz, dtype, n) <= parts * (row + 36) + (1 << 20)
