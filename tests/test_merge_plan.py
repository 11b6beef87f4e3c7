"""How sums and products of sparse operands are cut into partitions, from the host descriptors alone (no GPU): the
entries a partition holds at most tell which kernel a call takes."""
import ctypes

import pytest

from paper_2604_17198_amd import binding as nb

UNITS = 256                                    # compute units (what the library takes where there is no GPU)
ROUND = 4 * UNITS                              # workgroups that run at a time
SHORT, MIDDLE, LONG, WIDE = 1472, 4536, {nb.F32: 5544, nb.F64: 5040}, 3520

DENSE, COMPRESSED, NONUNIQUE, SINGLETON = nb.DENSE, nb.COMPRESSED, nb.NONUNIQUE, nb.SINGLETON
KINDS = {"vector": (COMPRESSED,), "csr": (DENSE, COMPRESSED), "dcsr": (COMPRESSED, COMPRESSED),
         "coo": (NONUNIQUE, SINGLETON), "csf3": (COMPRESSED, COMPRESSED, COMPRESSED)}
# extents that leave the row field of 32-bit keys room
EXTENTS = {"vector": (1 << 30,), "csr": (4000, 4000), "dcsr": (4000, 4000), "coo": (4000, 4000), "csf3": (60, 60, 60)}


def _operands(fmt, counts, extents):
    ops = (nb._Tensor * len(counts))()
    for op, n in zip(ops, counts):
        op.nlevels = len(KINDS[fmt])
        for m, (kind, extent) in enumerate(zip(KINDS[fmt], extents)):
            last = m == op.nlevels - 1
            op.lvl[m].kind, op.lvl[m].extent = kind, extent
            op.lvl[m].count = 0 if kind == DENSE else (n if last or fmt == "coo" else min(n, extent))
    return ops


def _split(total, k):
    return [total // k + (t < total % k) for t in range(k)]


def partitions(fmt, total, k, dtype, op=nb.OP_SPADD, extents=None, P=0):
    ops = _operands(fmt, _split(total, k), extents or EXTENTS[fmt])
    return int(nb.lib().nacho_num_partitions(op, ops, k, dtype, 0, P))


def needed(total, entries, k):
    return -(-total // (entries - k))


def whole_rounds(need):
    up = -(-need // ROUND) * ROUND
    return up if (up - need) * 12 <= need else need


def whole_units(need):
    return -(-need // UNITS) * UNITS


# (the last total that one round of long partitions holds, and the next)
ONE_ROUND_F64 = ROUND * (LONG[nb.F64] - nb.MAX_OPERANDS)


@pytest.mark.parametrize("k", [2, 3, 8])
@pytest.mark.parametrize("fmt,past", [("vector", MIDDLE), ("csf3", MIDDLE), ("csr", 5040), ("dcsr", 5040), ("coo", 5040)])
def test_doubles_past_a_round(fmt, past, k):
    """Ten places a thread as long as one round of such partitions holds the call; past it nine for vectors and tensors."""
    assert partitions(fmt, ONE_ROUND_F64, k, nb.F64) == whole_rounds(needed(ONE_ROUND_F64, 5040, k))
    for total in (ONE_ROUND_F64 + 1, 8_000_000, 12_345_679):
        assert partitions(fmt, total, k, nb.F64) == whole_rounds(needed(total, past, k)), total
    # floats have eleven
    assert partitions(fmt, ONE_ROUND_F64 + 1, k, nb.F32) == whole_rounds(needed(ONE_ROUND_F64 + 1, 5544, k))


# (the last total that one round of short partitions holds, and that five sixths of one do)
ONE_ROUND_SHORT = ROUND * (SHORT - nb.MAX_OPERANDS)
FIVE_SIXTHS = ROUND * 5 * (SHORT - nb.MAX_OPERANDS) // 6


def middle(fmt, total, k):
    """Partitions of a call of one round of middle ones: as many on every compute unit, but for coordinate lists."""
    need = needed(total, MIDDLE, k)
    return whole_rounds(need) if fmt == "coo" else whole_units(need)


TWO_A_UNIT = ROUND // 2 * (SHORT - nb.MAX_OPERANDS)
SPARSE_CSR, DENSE_CSR = (1_000_000, 4000), (4000, 4000)


@pytest.mark.parametrize("dtype", [nb.F32, nb.F64])
@pytest.mark.parametrize("fmt,extents,k,last", [
    ("vector", None, 2, TWO_A_UNIT), ("vector", None, 8, TWO_A_UNIT), ("csr", DENSE_CSR, 2, TWO_A_UNIT), ("csr", DENSE_CSR, 5, TWO_A_UNIT),
    ("csr", SPARSE_CSR, 2, ONE_ROUND_SHORT), ("csr", SPARSE_CSR, 8, ONE_ROUND_SHORT), ("dcsr", None, 2, FIVE_SIXTHS), ("dcsr", None, 8, FIVE_SIXTHS),
    ("coo", None, 2, FIVE_SIXTHS), ("coo", None, 4, FIVE_SIXTHS), ("coo", None, 5, ONE_ROUND_SHORT), ("coo", None, 8, ONE_ROUND_SHORT),
    ("csf3", None, 2, FIVE_SIXTHS), ("csf3", None, 8, FIVE_SIXTHS)])
def test_short_and_middle_partitions(fmt, extents, k, last, dtype):
    """The last call with short partitions and the first with middle ones, sums and products (not of tensors)."""
    for op in (nb.OP_SPADD,) if fmt == "csf3" else (nb.OP_SPADD, nb.OP_SPMUL):
        assert partitions(fmt, last, k, dtype, op, extents) == whole_rounds(needed(last, SHORT, k))
        assert partitions(fmt, last + 1, k, dtype, op, extents) == middle(fmt, last + 1, k)


@pytest.mark.parametrize("k", [2, 5])
@pytest.mark.parametrize("dtype", [nb.F32, nb.F64])
def test_csr_rows_of_16_entries(dtype, k):
    """Between two short partitions a compute unit and a round of them, the entries a row has in all operands decide."""
    total = 1_200_000
    assert partitions("csr", total, k, dtype, extents=(total // 16, 4000)) == middle("csr", total, k)
    assert partitions("csr", total, k, dtype, extents=(total // 16 + 1, 4000)) == whole_rounds(needed(total, SHORT, k))


# (the last total that one round of middle partitions holds; that two middle, that two long ones of floats a compute unit do)
ONE_ROUND_MIDDLE = ROUND * (MIDDLE - nb.MAX_OPERANDS)
TWO_MIDDLE, TWO_LONG = ONE_ROUND_MIDDLE // 2, ROUND // 2 * (LONG[nb.F32] - nb.MAX_OPERANDS)


@pytest.mark.parametrize("k", [2, 8])
@pytest.mark.parametrize("dtype", [nb.F32, nb.F64])
@pytest.mark.parametrize("fmt", list(EXTENTS))
def test_middle_and_long_partitions(fmt, dtype, k):
    assert partitions(fmt, ONE_ROUND_MIDDLE, k, dtype) == middle(fmt, ONE_ROUND_MIDDLE, k)
    total = ONE_ROUND_MIDDLE + 1
    assert partitions(fmt, total, k, dtype) == whole_rounds(needed(total, LONG[dtype], k))
    # two long partitions a compute unit instead of three middle ones: floats of CSR and DCSR
    long = dtype == nb.F32 and fmt in ("csr", "dcsr")
    for total, between in ((TWO_MIDDLE, False), (TWO_MIDDLE + 1, True), (TWO_LONG, True), (TWO_LONG + 1, False)):
        expected = whole_rounds(needed(total, LONG[dtype], k)) if long and between else middle(fmt, total, k)
        assert partitions(fmt, total, k, dtype) == expected, total


@pytest.mark.parametrize("dtype", [nb.F32, nb.F64])
@pytest.mark.parametrize("k", [2, 3, 8])
@pytest.mark.parametrize("extents", [(2000, 2000, 2000), (100_000, 40, 4000)])
def test_tensors_keep_short_keys_while_short_partitions_are_one_round(extents, k, dtype):
    """Where middle partitions span too many slices for 32-bit keys and short ones do not, short ones up to a whole round;
    tensors with few slices have middle ones from five sixths of a round on."""
    for total in (FIVE_SIXTHS, FIVE_SIXTHS + 1, 1_400_000, ONE_ROUND_SHORT):
        assert partitions("csf3", total, k, dtype, extents=extents) == whole_rounds(needed(total, SHORT, k)), total
    total = FIVE_SIXTHS + 1
    assert partitions("csf3", total, k, dtype, extents=(60, 60, 600)) == whole_units(needed(total, MIDDLE, k))
    # past the round
    past = partitions("csf3", ONE_ROUND_SHORT + 1, k, dtype, extents=extents)
    assert past in (needed(ONE_ROUND_SHORT + 1, WIDE, k), whole_units(needed(ONE_ROUND_SHORT + 1, MIDDLE, k)))


@pytest.mark.parametrize("dtype", [nb.F32, nb.F64])
@pytest.mark.parametrize("k", [2, 3, 8])
@pytest.mark.parametrize("fmt,extents", [(f, e) for f, e in EXTENTS.items()] +
                         [("dcsr", (800_000, 1_000_000)), ("coo", (400_000, 1_000_000)), ("csr", (400_000, 1_000_000)),
                          ("csf3", (2000, 2000, 2000)), ("csf3", (100_000, 40, 4000))])
def test_a_workspace_serves_operands_with_fewer_entries(fmt, extents, k, dtype):
    """Sized for the largest operands of a program, whatever partitions and keys the others take."""
    totals = [1, 1000, 700_000, 749_568, 749_569, 1_000_000, FIVE_SIXTHS, FIVE_SIXTHS + 1, ONE_ROUND_SHORT, ONE_ROUND_SHORT + 1, 2_000_000,
              2_700_000, 3_500_000, 4_200_000, 4_636_672, 4_636_673, 4_700_000, ONE_ROUND_F64, ONE_ROUND_F64 + 1, 5_669_000, 6_000_000,
              8_000_000, 10_800_000, 12_000_000, 20_000_000, 35_000_000]
    lib = nb.lib()
    parts, grain = nb._Parts(), ctypes.c_int64(0)
    for i, total in enumerate(totals):
        have = ctypes.c_size_t(0)
        assert lib.nacho_workspace_bytes(nb.OP_SPADD, _operands(fmt, _split(total, k), extents), k, dtype, 0, 0, ctypes.byref(have)) == 0
        for fewer in totals[:i + 1]:
            # (addresses are computed, nothing is read)
            rc = lib.nacho_workspace_parts(nb.OP_SPADD, _operands(fmt, _split(fewer, k), extents), k, dtype, 0, 0, 1 << 20, have.value,
                                           ctypes.byref(parts), ctypes.byref(grain), None)
            assert rc == 0, (total, fewer)
