"""How SpMV calls are cut and what workspace they ask for, from the host descriptors alone (no GPU)."""
import ctypes

import pytest

from paper_2604_17198_amd import binding as nb


def _operand(n_rows, nnz):
    t = nb._Tensor()
    t.nlevels = 2
    t.lvl[0].kind, t.lvl[0].extent = nb.DENSE, n_rows
    t.lvl[1].kind, t.lvl[1].extent, t.lvl[1].count = nb.COMPRESSED, 1000, nnz
    return ctypes.byref((nb._Tensor * 1)(t))


def _partitions(n_rows, nnz, dtype, P=0):
    return int(nb.lib().nacho_num_partitions(nb.OP_SPMV, _operand(n_rows, nnz), 1, dtype, 0, P))


def _workspace(n_rows, nnz, dtype, P=0):
    size = ctypes.c_size_t(0)
    assert nb.lib().nacho_workspace_bytes(nb.OP_SPMV, _operand(n_rows, nnz), 1, dtype, 0, P, ctypes.byref(size)) == 0
    return size.value


@pytest.mark.parametrize("nnz,n_rows,dtype,grain", [
    (1_399_999, 100, nb.F32, 512), (1_400_000, 100, nb.F32, 1024),
    (4_800_000, 100_000, nb.F32, 1024), (4_800_000, 100_001, nb.F32, 512), (2**31 - 1, 1000, nb.F32, 1024),
    (1_399_999, 100, nb.F64, 512), (4_800_000, 100_000, nb.F64, 512), (4_800_000, 100_001, nb.F64, 512)])
def test_partitions_are_long_where_rows_are(nnz, n_rows, dtype, grain):
    """Floats: 1024 non-zeros from 1.4M of them and 48 a row on, else 512; doubles 512."""
    assert _partitions(n_rows, nnz, dtype) == -(-nnz // grain)


@pytest.mark.parametrize("dtype,capacity", [(nb.F32, 1024), (nb.F64, 512)])
def test_the_callers_count_is_kept_as_long_as_partitions_fit(dtype, capacity):
    for n_rows in (100, 1_000_000):
        assert _partitions(n_rows, 1000 * capacity, dtype, 1000) == 1000
        assert _partitions(n_rows, 1000 * capacity + 1, dtype, 1000) == 1001
        assert _partitions(n_rows, 5_000_000, dtype, 1) == -(-5_000_000 // capacity)


@pytest.mark.parametrize("dtype", [nb.F32, nb.F64])
def test_a_workspace_serves_matrices_with_fewer_non_zeros(dtype):
    """Whatever their rows: what a call needs is the size for as many partitions as it has, given as P."""
    for nnz in (1000, 1_399_999, 1_400_000, 1_500_000, 5_000_000, 50_000_000):
        have = _workspace(100, nnz, dtype)
        assert have == _workspace(10_000_000, nnz, dtype)
        for fewer in (nnz, nnz - 1, nnz // 2 + 1, 1_399_999):
            for n_rows in (100, 10_000_000):
                if fewer <= nnz:
                    assert _workspace(n_rows, fewer, dtype, _partitions(n_rows, fewer, dtype)) <= have
