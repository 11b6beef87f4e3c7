"""GPU parity of SpMM calls that sort their partitions by column (from 600 MB of gathers on, B larger than an L2), and of those
that deal out the partitions of long rows: at every grain, in two passes, with empty rows, one row with most of the non-zeros,
rows that end with a partition, a matrix without long rows, and a workspace that has no room for the sort."""
import numpy as np
import pytest
import torch

import oracle
from paper_2604_17198_amd import binding as nb
from gpu_util import csr_operand, dev
from util import tol_ok

pytestmark = pytest.mark.gpu

TOL = {np.float32: 1e-5, np.float64: 1e-12}


def _matrix(rng, lens, n_cols, dtype):
    """A CSR matrix with the given row lengths: evenly spaced columns from a random place on."""
    lens = np.asarray(lens, dtype=np.int64)
    pos = np.zeros(len(lens) + 1, np.int32)
    pos[1:] = np.cumsum(lens)
    row = np.repeat(np.arange(len(lens)), lens)
    at = np.arange(int(pos[-1])) - pos[row]
    step = np.maximum(n_cols // np.maximum(lens, 1), 1)
    start = rng.integers(0, np.maximum(n_cols - step * (lens - 1), 1))
    return {"n_rows": len(lens), "n_cols": n_cols, "pos": pos, "crd": (start[row] + at * step[row]).astype(np.int32),
            "val": rng.uniform(-1, 1, len(row)).astype(dtype)}


def _lengths(rng, kind, nnz, n_cols):
    if kind == "long":                                  # rows of many partitions, empty ones between, short ones behind
        lens = np.concatenate([np.full(10, n_cols // 2), np.zeros(50), np.full(20, 64 * 192), rng.integers(0, 9, 4000)])
    elif kind == "one":                                 # one row holds all it can
        lens = np.concatenate([np.full(700, 3), [n_cols], np.zeros(5)])
    else:                                               # "short": no partition lies inside one row
        lens = np.full(200, 9)
    lens = lens.astype(np.int64)
    left = nnz - int(lens.sum())
    assert left >= 0
    return np.concatenate([lens, np.full(left // 40, 40), [left % 40]]).astype(np.int64)


# (row of B in bytes: below 144, 192, 384 and 768, and above; non-zeros enough for 600 MB)
@pytest.mark.parametrize("kind,dtype,n,nnz", [("long", np.float32, 33, 4_700_000), ("long", np.float64, 18, 4_200_000),
                                              ("short", np.float32, 37, 4_100_000), ("one", np.float64, 48, 1_600_000),
                                              ("long", np.float64, 101, 760_000), ("one", np.float32, 300, 520_000)])
def test_sorted_partitions(kind, dtype, n, nnz):
    rng = np.random.default_rng(n)
    item = np.dtype(dtype).itemsize
    n_cols = 60_000
    A = _matrix(rng, _lengths(rng, kind, nnz, n_cols), n_cols, dtype)
    op, code = csr_operand(A), nb.F64 if dtype == np.float64 else nb.F32
    B = rng.uniform(-1, 1, (n_cols, n)).astype(dtype)
    grain = 64 if n * item >= 768 else 128 if n * item >= 384 else 192 if n * item >= 144 else 256
    big = nb.workspace_bytes(nb.OP_SPMM, [op], code, n)
    ref, sabs = oracle.spmm(A["pos"], A["crd"], A["val"], B)
    for size in (big, big - 1):                         # (one byte short: unsorted)
        print(f"spmm sorted {kind} n={n} nnz={nnz} ws={size}", flush=True)
        ws = torch.full((size,), 0xff, dtype=torch.uint8, device="cuda")
        C = torch.full((A["n_rows"], n), float("nan"), dtype=dev(B).dtype, device="cuda")
        nb.nacho_spmm(op, dev(B), C, ws=ws)
        assert tol_ok(C.cpu().numpy(), ref, sabs, TOL[dtype]).all(), (kind, n, size)
        t = nb.workspace_parts(nb.OP_SPMM, [op], code, ws, n)
        assert (t["grain"] == grain * n) == (size == big)
        queries = np.minimum(np.arange(t["P"] + 1, dtype=np.int64) * (t["grain"] // n), nnz)
        table = oracle.partition([oracle.csr(A["pos"], A["crd"], A["n_rows"], n_cols)], t["P"], queries=queries)
        assert np.array_equal(t["posn"].cpu().numpy().astype(np.int64), table["posn"])
        assert np.array_equal(t["cost"].cpu().numpy(), table["cost"] * n)


@pytest.mark.parametrize("n", [4, 5, 64, 65])
def test_rows_dealt_out(n):
    """Rows of 3 to 40 whole partitions of 64, starting and ending inside one or with one; B larger than an L2."""
    rng = np.random.default_rng(n)
    n_cols = 4_200_000 // (4 * n) + 1
    lens = [64 * 3, 64 * 4, 64 * 5, 64 * 9 + 1, 63, 64 * 40, 0, 0, 17, 64 * 12 - 1, 64 * 8, 64 * 16 + 40, 1]
    A = _matrix(rng, [min(l, n_cols) for l in lens * 5], n_cols, np.float32)
    B = rng.uniform(-1, 1, (n_cols, n)).astype(np.float32)
    op = csr_operand(A)
    ws = torch.empty(nb.workspace_bytes(nb.OP_SPMM, [op], nb.F32, n), dtype=torch.uint8, device="cuda")
    C = nb.nacho_spmm(op, dev(B), ws=ws)
    ref, sabs = oracle.spmm(A["pos"], A["crd"], A["val"], B)
    assert tol_ok(C.cpu().numpy(), ref, sabs, 1e-5).all()
    t = nb.workspace_parts(nb.OP_SPMM, [op], nb.F32, ws, n)
    nnz = int(A["pos"][-1])
    queries = np.minimum(np.arange(t["P"] + 1, dtype=np.int64) * (t["grain"] // n), nnz)
    table = oracle.partition([oracle.csr(A["pos"], A["crd"], A["n_rows"], n_cols)], t["P"], queries=queries)
    assert np.array_equal(t["coord"].cpu().numpy().astype(np.int64), table["coord"])
    assert np.array_equal(t["posn"].cpu().numpy().astype(np.int64), table["posn"])


def _records(fn, n_records):
    """The wavefront records of one call through the instrumented library."""
    nb.select_library(True)
    try:
        rec = torch.zeros(n_records * np.dtype(nb.WAVE_RECORD).itemsize, dtype=torch.uint8, device="cuda")
        nb.instrument(rec)
        fn()
        torch.cuda.synchronize()
        nb.instrument(None)
    finally:
        nb.select_library(False)
    return rec.cpu().numpy().view(np.dtype(nb.WAVE_RECORD))


@pytest.mark.parametrize("dtype,n,nnz,grain,join", [(np.float32, 200, 800_003, 64, 4), (np.float64, 97, 1_000_001, 64, 4),
                                                    (np.float32, 100, 2_200_000, 128, 4), (np.float64, 300, 810_000, 64, 4)])
@pytest.mark.parametrize("kind", ["random", "wide", "band", "long"])
def test_partitions_joined(kind, dtype, n, nnz, grain, join):
    """Short rows with columns at random: every wavefront executes `join` partitions of the table in one piece (one long row
    among them, of more joined partitions than one group of the fix-up adds; empty rows), also where rows hold a partition that
    covers most of the columns.  In a narrow band, or with long rows: one each.  The table is that of the short partitions."""
    rng = np.random.default_rng(n)
    n_cols = 50_000
    head = [0, 7, grain * join * 40 + 5, 0, 0, grain * join, 1] if kind != "long" else [n_cols // 2] * 16 + [0, 3]
    left = nnz - sum(head)
    each = grain * 3 // 2 if kind == "wide" else 30
    lens = np.array(head + [each] * (left // each) + [left % each, 0], np.int64)
    A = _matrix(rng, lens, n_cols, dtype)
    if kind in ("random", "band"):                      # the columns of rows of 30: anywhere, or in a band along the diagonal
        row = np.repeat(np.arange(len(lens)), lens)
        short = lens[row] <= 30
        place = rng.integers(0, n_cols, len(row)) if kind == "random" else (row * (n_cols - 2000) // len(lens)
                                                                            + rng.integers(0, 2000, len(row)))
        key = np.where(short, row * n_cols + place, row * n_cols + A["crd"])
        key = np.unique(key)
        row, A["crd"] = key // n_cols, (key % n_cols).astype(np.int32)
        A["pos"][1:] = np.cumsum(np.bincount(row, minlength=len(lens)))
        A["val"] = A["val"][:len(key)]
    nnz = int(A["pos"][-1])
    op, code = csr_operand(A), nb.F64 if dtype == np.float64 else nb.F32
    B = rng.uniform(-1, 1, (n_cols, n)).astype(dtype)
    ref, sabs = oracle.spmm(A["pos"], A["crd"], A["val"], B)
    ws = torch.full((nb.workspace_bytes(nb.OP_SPMM, [op], code, n),), 0xff, dtype=torch.uint8, device="cuda")
    C = torch.full((A["n_rows"], n), float("nan"), dtype=dev(B).dtype, device="cuda")
    print(f"spmm joined {kind} n={n} nnz={nnz}", flush=True)
    nb.nacho_spmm(op, dev(B), C, ws=ws)
    assert tol_ok(C.cpu().numpy(), ref, sabs, TOL[dtype]).all()
    t = nb.workspace_parts(nb.OP_SPMM, [op], code, ws, n)
    P = t["P"]
    assert t["grain"] == grain * n and P == -(-nnz // grain)
    queries = np.minimum(np.arange(P + 1, dtype=np.int64) * grain, nnz)
    table = oracle.partition([oracle.csr(A["pos"], A["crd"], A["n_rows"], n_cols)], P, queries=queries)
    assert np.array_equal(t["coord"].cpu().numpy().astype(np.int64), table["coord"])
    assert np.array_equal(t["posn"].cpu().numpy().astype(np.int64), table["posn"])
    items = _records(lambda: nb.nacho_spmm(op, dev(B), C, ws=ws), P)["items"].astype(np.int64)
    assert tol_ok(C.cpu().numpy(), ref, sabs, TOL[dtype]).all()
    assert items.sum() == nnz
    each = grain * (join if kind in ("random", "wide") else 1)
    assert np.count_nonzero(items) == -(-nnz // each) and items.max() == each
