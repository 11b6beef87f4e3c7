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
