"""Matrices of 2^31 - 1 rows, the most there are: a row and the rows a wavefront looks at behind it may lie past what 32 bits with a
sign hold.  Values are small whole numbers, so that every sum is exact in any order; rows nothing is stored in are exactly 0."""
import numpy as np
import pytest
import torch

from paper_2604_17198_amd import binding as nb
from gpu_util import dev

pytestmark = pytest.mark.gpu

ROWS = 2**31 - 1
COLS = 4000
DTYPES = [np.float32, np.float64]
# where the stored rows lie and how many non-zeros they have: one partition that spans all rows, and a few
WHERE = {"first, one partition": {0: 5, 3: 60, 4: 1, 700: 200}, "first, several": {0: 900, 1: 1, 2: 47, 3: 3000, 5000: 48},
         "last, one partition": {ROWS - 701: 5, ROWS - 513: 60, ROWS - 64: 1, ROWS - 1: 200},
         "the last": {ROWS - 1: 3000}, "last, several": {ROWS - 2000: 900, ROWS - 63: 48, ROWS - 2: 3, ROWS - 1: 700},
         "both ends": {2: 47, 2**30: 900, ROWS - 1030: 1, ROWS - 600: 2500, ROWS - 512: 3, ROWS - 1: 30}}


def _tall(lens, dtype):
    """(the operand, its entries as arrays): the given rows of ROWS."""
    rng = np.random.default_rng(len(lens))
    rows = sorted(lens)
    pos = torch.zeros(ROWS + 1, dtype=torch.int32, device="cuda")
    stored = 0
    for r, behind in zip(rows, rows[1:] + [ROWS]):
        stored += lens[r]
        pos[r + 1:behind + 1] = stored
    crd = np.concatenate([np.sort(rng.choice(COLS, lens[r], replace=False)) for r in rows]).astype(np.int32)
    val = rng.integers(1, 9, len(crd)).astype(dtype)
    op = nb.csr(pos, dev(crd), ROWS, COLS, dev(val))
    return op, np.repeat(np.arange(len(rows)), [lens[r] for r in rows]), np.array(rows), crd, val


def _expect(got, rows, want, tag):
    torch.cuda.synchronize()
    at = torch.from_numpy(rows).to("cuda")
    assert np.array_equal(got[at].cpu().numpy(), want), tag
    assert int(torch.count_nonzero(got)) == int(np.count_nonzero(want)), tag       # (NaN counts: a row never written)


def _spmv_forms():
    return {"P=0": lambda op, x, y: nb.nacho_spmv(op, x, y), "P=3": lambda op, x, y: nb.nacho_spmv(op, x, y, P=3),
            "static": lambda op, x, y: nb.nacho_spmv_static(op, x, y),
            "fused": lambda op, x, y: nb.nacho_spmv_fused(op, x, y)}


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("where", list(WHERE))
def test_spmv(where, dtype):
    op, of_row, rows, crd, val = _tall(WHERE[where], dtype)
    x = np.random.default_rng(9).integers(1, 9, COLS).astype(dtype)
    want = np.zeros(len(rows), dtype)
    np.add.at(want, of_row, val * x[crd])
    y = torch.empty(ROWS, dtype=dev(x).dtype, device="cuda")
    for tag, call in _spmv_forms().items():
        print(f"tall spmv {where} {np.dtype(dtype).name} {tag}", flush=True)
        y.fill_(float("nan"))
        call(op, dev(x), y)
        _expect(y, rows, want, tag)


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("where", list(WHERE))
def test_spmm(where, dtype):
    op, of_row, rows, crd, val = _tall(WHERE[where], dtype)
    for n in (1, 2):
        B = np.random.default_rng(9).integers(1, 9, (COLS, n)).astype(dtype)
        want = np.zeros((len(rows), n), dtype)
        np.add.at(want, of_row, val[:, None] * B[crd])
        for P in (0, 3):
            print(f"tall spmm {where} {np.dtype(dtype).name} n={n} P={P}", flush=True)
            C = torch.full((ROWS, n), float("nan"), dtype=dev(B).dtype, device="cuda")
            nb.nacho_spmm(op, dev(B), C, P=P)
            _expect(C, rows, want, (n, P))
            del C


def _rows_of(pos):
    """The row of every entry, from a pos array on the GPU (as it has so many rows, in stretches)."""
    found = []
    for r in range(0, ROWS, 1 << 28):
        part = pos[r:min(r + (1 << 28), ROWS) + 1]
        lens = part[1:] - part[:-1]
        at = torch.nonzero(lens)[:, 0]
        found.append(torch.repeat_interleave(at + r, lens[at].long()))
    return torch.cat(found)


def _csr_of(keys, val):
    """A matrix of ROWS rows from its entries (row * COLS + column, ascending), on the GPU."""
    rows = keys // COLS
    pos = torch.empty(ROWS + 1, dtype=torch.int32, device="cuda")
    for r in range(0, ROWS + 1, 1 << 27):
        part = torch.arange(r, min(r + (1 << 27), ROWS + 1), device="cuda")
        pos[r:r + len(part)] = torch.searchsorted(rows, part, out_int32=True)
    return nb.csr(pos, (keys % COLS).to(torch.int32), ROWS, COLS, val)


# spread: entries of every operand all over the rows (none: one partition that spans all of them); end: in the last rows
@pytest.mark.parametrize("name,operands,spread,end", [("spadd", 2, 3_000_000, 500_000), ("spmul", 2, 3_000_000, 500_000),
                                                      ("spadd", 4, 1_500_000, 40_000), ("spmul", 4, 1_500_000, 40_000),
                                                      ("spadd", 2, 0, 400)])
def test_sums_and_products(name, operands, spread, end):
    """Operands that share half of their entries; partitions start and end in the last rows."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(spread + operands)
    some = lambda lo, hi, n: torch.randint(lo, hi, (n,), dtype=torch.int64, device="cuda", generator=gen)
    entries = lambda first, n: some(first, ROWS, n) * COLS + some(0, COLS, n)
    common = torch.cat([entries(0, spread // 2), entries(ROWS - 700, end // 2)])
    ops, keys, vals = [], [], []
    for t in range(operands):
        keys.append(torch.unique(torch.cat([common, entries(0, spread // 2), entries(ROWS - 70, end // 2)])))
        vals.append(some(1, 9, len(keys[t])).to(torch.float32))
        ops.append(_csr_of(keys[t], vals[t]))
    every, place, times = torch.unique(torch.cat(keys), return_inverse=True, return_counts=True)
    if name == "spadd":
        want = torch.zeros(len(every), dtype=torch.float32, device="cuda").index_add_(0, place, torch.cat(vals))
    else:
        want = torch.ones(len(every), dtype=torch.float32, device="cuda")
        for k, v in zip(keys, vals):
            want[torch.searchsorted(every, k)] *= v
        every, want = every[times == operands], want[times == operands]
    print(f"tall {name} {operands} operands, {len(every)} entries", flush=True)
    out = nb.SparseOut("csr", 0, len(every), torch.float32, "cuda", n_rows=ROWS)
    (nb.nacho_spadd_k if name == "spadd" else nb.nacho_spmul_k)(ops, out)
    torch.cuda.synchronize()
    assert int(out.status[0]) == 0 and out.counts[:2].tolist() == [ROWS, len(every)]
    assert int(out.pos1[0]) == 0 and int(out.pos1[ROWS]) == len(every)
    assert torch.equal(_rows_of(out.pos1), every // COLS)
    assert torch.equal(out.crd1[:len(every)].long(), every % COLS) and torch.equal(out.val[:len(every)], want)
