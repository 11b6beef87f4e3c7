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


# (row of B in bytes; the first number of columns that sorts; non-zeros of a sorted and an unsorted partition)
@pytest.mark.parametrize("dtype,n,n_cols,nnz,short,long", [(nb.F32, 16, 121_875, 10_000_000, 256, 512),
                                                           (nb.F32, 64, 30_469, 3_000_000, 192, 512),
                                                           (nb.F32, 96, 26_042, 2_500_000, 128, 512),
                                                           (nb.F64, 200, 6_250, 1_000_000, 64, 256)])
def test_b_that_two_l2s_hold_is_not_sorted_for(dtype, n, n_cols, nnz, short, long):
    assert _partitions(n_cols, nnz, dtype, n) == -(-nnz // short)
    assert _partitions(n_cols - 1, nnz, dtype, n) == -(-nnz // long)
