"""GPU parity at the edges of the kernels' tiles and of the rules that choose a kernel: column counts around the pieces
and lanes of SpMM, row lengths around SpMV's long rows, calls just under and over the sizes at which a partition kernel
or the long partitions of a merge come in, rows that do not fit a merge key's row field, and more workgroups than one
look-back step reads.  Index arrays and boundaries bit-exact; values as the oracle has them, within the tolerances of
the files whose checks are used here."""
import numpy as np
import pytest
import torch

import oracle
import test_gpu_coo as coo
import test_gpu_csf3 as csf3
import test_gpu_partition as part
import test_gpu_spadd as add
import test_gpu_spmm as spmm
import test_gpu_spmul as mul
import test_gpu_spmul_dcsr as mul_dcsr
import test_gpu_spmv as spmv
from paper_2604_17198_amd import binding as nb
from gpu_util import csr_operand, dev, parts_to_numpy
from util import to_csr, tol_ok

pytestmark = pytest.mark.gpu

DTYPES = [np.float32, np.float64]
UNITS = 256                                     # compute units; a merge keeps 4 workgroups on each


def _matrix(rng, lens, n_cols, dtype):
    """A CSR matrix with the given row lengths."""
    lens = np.asarray(lens)
    crd = np.concatenate([np.sort(rng.choice(n_cols, l, replace=False)) for l in lens] + [np.zeros(0, np.int64)])
    pos = np.zeros(len(lens) + 1, np.int32)
    pos[1:] = np.cumsum(lens)
    return {"n_rows": len(lens), "n_cols": n_cols, "pos": pos, "crd": crd.astype(np.int32),
            "val": rng.uniform(-1, 1, len(crd)).astype(dtype)}


# ---- SpMM -------------------------------------------------------------------
@pytest.mark.parametrize("dtype", DTYPES)
def test_spmm_columns(dtype):
    """One piece of a row (16 bytes), a lane group's width (4, 8, 16 lanes), 1 to 4 pieces a lane, two passes -- and one
    column on either side of each; with a partition kernel and without one."""
    rng = np.random.default_rng(1)
    v = 16 // np.dtype(dtype).itemsize
    A = _matrix(rng, [0, 300, 0, 0, 1, 900, 3, 5, 0, 64, 63, 65, 0], 1000, dtype)
    edges = {1, 2, 3} | {v * lanes * pieces + d for lanes, pieces in ((1, 1), (4, 1), (8, 1), (16, 1), (16, 2), (16, 3), (16, 4))
                         for d in (-1, 0, 1)} | {257, 300}
    for n in sorted(e for e in edges if e > 0):
        B = rng.uniform(-1, 1, (A["n_cols"], n)).astype(dtype)
        for P in (0, 9):
            spmm._check(A, B, P, "columns")


@pytest.mark.parametrize("nnz", [1, 63, 64, 65, 262_144, 262_145, 2_097_151, 2_097_153])
def test_spmm_grain(nnz):
    """Partitions of 64 non-zeros up to 64 x 4096 of them, of 512 from 512 x 4096 on; rows of a few entries, one that
    spans many partitions, and a run of carries either side of what one group adds by itself (32)."""
    rng = np.random.default_rng(nnz)
    n_rows, n_cols = max(1, nnz // 9), 40_000
    lens = np.full(n_rows, nnz // n_rows)
    lens[-1] += nnz - lens.sum()
    if nnz > 60_000:
        for r, l in ((n_rows // 2, 64 * 32), (n_rows // 3, 64 * 34), (7, 20_000)):
            take = np.flatnonzero(lens > 1)[:l]
            lens[take] -= 1
            lens[r] += len(take)
    starts = rng.integers(0, n_cols - int(lens.max()), n_rows)
    pos = np.zeros(n_rows + 1, np.int32)
    pos[1:] = np.cumsum(lens)
    crd = (np.repeat(starts, lens) + np.arange(nnz) - np.repeat(pos[:-1], lens)).astype(np.int32)
    A = {"n_rows": n_rows, "n_cols": n_cols, "pos": pos, "crd": crd, "val": rng.uniform(-1, 1, nnz).astype(np.float32)}
    spmm._check(A, rng.uniform(-1, 1, (n_cols, 5)).astype(np.float32), 0, "grain")


@pytest.mark.parametrize("extra", [0, 1])
def test_spmm_rows_per_partition(extra):
    """1024 rows a partition: with more the partition kernel writes the zeros of empty rows."""
    rng = np.random.default_rng(5)
    lens = np.zeros(2 * 1024 + extra, np.int64)         # two partitions of 64 non-zeros
    lens[[3, 700, 1500]] = 50, 30, 20
    A = _matrix(rng, lens, 500, np.float64)
    spmm._check(A, rng.uniform(-1, 1, (500, 6)), 0, "rows per partition")


def test_spmm_workspace_for_fewer_columns():
    """A workspace sized without a column count (64 of them) serves 200 columns, and its table can be read."""
    rng = np.random.default_rng(6)
    A = _matrix(rng, [0, 300, 0, 0, 1, 900, 3, 5, 0, 64], 1000, np.float32)
    op = csr_operand(A)
    B = rng.uniform(-1, 1, (1000, 200)).astype(np.float32)
    ws = torch.empty(nb.workspace_bytes(nb.OP_SPMM, [op], nb.F32), dtype=torch.uint8, device="cuda")
    assert ws.numel() < nb.workspace_bytes(nb.OP_SPMM, [op], nb.F32, 200)
    C = nb.nacho_spmm(op, dev(B), ws=ws)
    table = nb.workspace_parts(nb.OP_SPMM, [op], nb.F32, ws, 200)
    ref, sabs = oracle.spmm(A["pos"], A["crd"], A["val"], B)
    assert tol_ok(C.cpu().numpy(), ref, sabs, spmm.TOL[np.float32]).all()
    assert int(table["posn"][-1, 0, 1]) == int(A["pos"][-1])


# ---- SpMV -------------------------------------------------------------------
@pytest.mark.parametrize("dtype", DTYPES)
def test_spmv_row_lengths(dtype):
    """Rows around the four products a lane adds at a time, the 48 from which a wavefront adds them, and the partition."""
    rng = np.random.default_rng(11)
    lens = [1, 2, 3, 4, 5, 7, 8, 9, 0, 46, 47, 48, 49, 50, 63, 64, 65, 0, 0]
    for grain in (512,) if dtype == np.float64 else (512, 1024):       # (floats: 1024 for a caller's P)
        lens += [grain - 1, grain, grain + 1, 3 * grain]
    A = _matrix(rng, lens * 3, 4000, dtype)
    x = rng.uniform(-1, 1, 4000).astype(dtype)
    for P in (0, 5):
        spmv._check(A, x, P, "row lengths")


@pytest.mark.parametrize("parts,rows,cols", [
    (1024, 5000, 3000), (1025, 5000, 600_000), (1025, 5000, 524_288), (1025, 5000, 524_289),
    (8192, 5000, 3000), (8193, 5000, 3000), (100, 1 << 17, 3000), (100, (1 << 17) + 1, 3000)])
def test_spmv_calls_without_a_partition_kernel(parts, rows, cols):
    """Partitions, the bytes of x and rows around the limits up to which the wavefronts search their own rows: the
    stored table is Algorithm 1's either way."""
    rng = np.random.default_rng(parts + rows + cols)
    nnz = parts * 512 - 100
    lens = np.zeros(rows, np.int64)
    some = np.sort(rng.choice(rows, min(rows, 4000), replace=False))
    lens[some] = nnz // len(some)
    lens[some[:nnz % len(some)]] += 1
    pos = np.zeros(rows + 1, np.int32)
    pos[1:] = np.cumsum(lens)
    # (columns of a row: evenly spaced over the row of A)
    at = np.arange(nnz) - np.repeat(pos[:-1].astype(np.int64), lens)
    crd = (at * cols // np.repeat(np.maximum(lens, 1), lens)).astype(np.int32)
    A = {"n_rows": rows, "n_cols": cols, "pos": pos, "crd": crd, "val": rng.uniform(-1, 1, nnz)}
    x = rng.uniform(-1, 1, cols)
    spmv._check(A, x, 0, "limits")
    op = csr_operand(A)
    ws = torch.empty(nb.workspace_bytes(nb.OP_SPMV, [op], nb.F64), dtype=torch.uint8, device="cuda")
    nb.nacho_spmv(op, dev(x), ws=ws)
    t = nb.workspace_parts(nb.OP_SPMV, [op], nb.F64, ws)
    queries = np.minimum(np.arange(t["P"] + 1, dtype=np.int64) * 512, nnz)
    ref = oracle.partition([oracle.csr(pos, crd, rows, cols)], t["P"], queries=queries)
    got = {k: v.cpu().numpy() for k, v in t.items() if k in ("coord", "posn", "cost")}
    part._compare(got, ref, "limits")


@pytest.mark.parametrize("grain,parts,rows,cols,search", [
    (512, 2048, 5000, (1 << 20) + 1, False), (512, 2049, 5000, (1 << 20) + 1, True), (512, 2049, 5000, 1 << 20, False),
    (512, 10240, 120_000, 3000, False), (512, 10241, 120_000, 3000, True), (512, 3, 512, 3000, False), (512, 3, 513, 3000, True),
    (1024, 1400, 5000, 1 << 20, False), (1024, 1400, 5000, (1 << 20) + 1, True),
    (1024, 8192, 5000, 3000, False), (1024, 8193, 5000, 3000, True), (1024, 8192, 1 << 17, 3000, False), (1024, 8192, (1 << 17) + 1, 3000, True)])
def test_spmv_of_floats_without_a_partition_kernel(grain, parts, rows, cols, search):
    """The same for floats, whose short partitions count half, and whose partitions are long where rows are."""
    rng = np.random.default_rng(parts + rows + cols)
    nnz = parts * grain - 100
    lens = np.zeros(rows, np.int64)
    some = np.sort(rng.choice(rows, min(rows, 4000), replace=False))
    lens[some] = nnz // len(some)
    lens[some[:nnz % len(some)]] += 1
    pos = np.zeros(rows + 1, np.int32)
    pos[1:] = np.cumsum(lens)
    at = np.arange(nnz) - np.repeat(pos[:-1].astype(np.int64), lens)
    crd = (at * cols // np.repeat(np.maximum(lens, 1), lens)).astype(np.int32)
    A = {"n_rows": rows, "n_cols": cols, "pos": pos, "crd": crd, "val": rng.uniform(-1, 1, nnz).astype(np.float32)}
    x = rng.uniform(-1, 1, cols).astype(np.float32)
    nb.profile_enable(True)
    try:
        spmv._check(A, x, 0, "limits of floats")
        kernels = [name for name, _ in nb.profile_read()]
    finally:
        nb.profile_enable(False)
    assert ("partition" in kernels) == search
    op = csr_operand(A)
    ws = torch.empty(nb.workspace_bytes(nb.OP_SPMV, [op], nb.F32), dtype=torch.uint8, device="cuda")
    nb.nacho_spmv(op, dev(x), ws=ws)
    t = nb.workspace_parts(nb.OP_SPMV, [op], nb.F32, ws)
    assert t["P"] == parts and t["grain"] == grain
    queries = np.minimum(np.arange(t["P"] + 1, dtype=np.int64) * grain, nnz)
    ref = oracle.partition([oracle.csr(pos, crd, rows, cols)], t["P"], queries=queries)
    got = {k: v.cpu().numpy() for k, v in t.items() if k in ("coord", "posn", "cost")}
    part._compare(got, ref, "limits of floats")


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("parts,rows", [(1, 256), (1, 257), (3, 768), (3, 769), (1, 1 << 17), (512, 1 << 17), (512, (1 << 17) + 1)])
@pytest.mark.parametrize("first", [0, 0.5, 1])
def test_spmv_rows_per_partition(parts, rows, first, dtype):
    """All non-zeros at the first, the middle or the last rows: no wavefront is left with the zeros of more than 256 of the
    others, with more rows a partition kernel writes them."""
    rng = np.random.default_rng(parts + rows)
    grain = 512 if dtype == np.float64 else 1024
    nnz, full = parts * grain - 7, max(1, parts // 4)
    lens = np.full(full, nnz // full)
    lens[0] += nnz - lens.sum()
    r0 = int(first * (rows - full))
    A = _matrix(rng, np.concatenate([np.zeros(r0, np.int64), lens, np.zeros(rows - full - r0, np.int64)]), 9000, dtype)
    nb.profile_enable(True)
    try:
        spmv._check(A, rng.uniform(-1, 1, 9000).astype(dtype), 0, "rows per partition")
        kernels = [name for name, _ in nb.profile_read()]
    finally:
        nb.profile_enable(False)
    assert ("partition" in kernels) == (rows > min(256 * parts, 1 << 17))


# ---- partition search ---------------------------------------------------------
def test_partition_two_vectors():
    """Two operands are searched by splits of the merge path: lengths and spreads far apart, ties, nothing interleaved."""
    rng = np.random.default_rng(21)
    draw = lambda lo, hi, n: np.unique(rng.integers(lo, hi, n)).astype(np.int32)
    tied = draw(0, 1 << 30, 200_000)
    cases = {"equal": (draw(0, 1 << 30, 300_000), draw(0, 1 << 30, 300_000)), "tied": (tied, tied.copy()),
             "one": (draw(0, 1 << 30, 300_000), np.array([1 << 29], np.int32)),
             "apart": (draw(0, 1 << 20, 100_000), draw(1 << 20, 1 << 30, 100_000)),
             "behind": (draw(1 << 29, 1 << 30, 70_000), draw(0, 1 << 29, 1000)),
             "empty": (np.zeros(0, np.int32), draw(0, 1 << 30, 5000))}
    for name, vs in cases.items():
        for order in (vs, vs[::-1]):
            g, o = part._vec_ops(order, (1 << 30) + 7)
            for P in (3, 64, 3000):
                print(f"partition two vectors {name} sizes={[len(v) for v in order]} P={P}", flush=True)
                part._compare(parts_to_numpy(nb.nacho_partition(g, P)), oracle.partition(o, P), (name, P))


# ---- merge --------------------------------------------------------------------
def _short_limit(dtype):
    """Most entries of vectors in short partitions: two a compute unit (1512 places, less 64 words around runs)."""
    return UNITS * 2 * (min(3 * 504, 3 * 512 - 64) - 8)


@pytest.mark.parametrize("k", [2, 3])
@pytest.mark.parametrize("over", [0, 1])
def test_merge_short_and_middle_partitions(k, over):
    rng = np.random.default_rng(31)
    for dtype in DTYPES:
        total = _short_limit(dtype) + over
        sizes = [total // k] * (k - 1)
        sizes.append(total - sum(sizes))
        vs = [np.sort(rng.choice(1 << 22, n, replace=False)).astype(np.int32) for n in sizes]
        add.check_vec(vs, [rng.uniform(-1, 1, n).astype(dtype) for n in sizes], 1 << 22, 0, f"limit+{over}")


@pytest.mark.parametrize("per_unit,places", [(2, 3), (4, 9)])
@pytest.mark.parametrize("over", [0, 1])
@pytest.mark.parametrize("dtype", DTYPES)
def test_merge_between_lengths_of_partitions(per_unit, places, over, dtype):
    """The lines between short, middle and long partitions, from both sides: the sum and the product are those of the same
    call in other partitions (vectors: the shared tests hold the oracle's), bit for bit."""
    total = UNITS * per_unit * (min(places * 504, places * 512 - 64) - 8) + over
    gen = torch.Generator(device="cuda").manual_seed(total)
    as_torch = torch.float64 if dtype == np.float64 else torch.float32
    ops = []
    for n in (total - total // 3, total // 3):
        keys = torch.cumsum(torch.randint(1, 3, (n,), device="cuda", generator=gen), 0).to(torch.int32)
        ops.append(nb.vector(keys, (1 << 30) + 7, torch.rand(n, device="cuda", generator=gen, dtype=as_torch)))
    print(f"lengths of partitions {total} {dtype.__name__}", flush=True)
    for call in (nb.nacho_spadd_k, nb.nacho_spmul_k):
        a, b = (call(ops, nb.SparseOut("vector", 0, total, as_torch, "cuda"), P=P) for P in (0, 2500))
        n = int(a.counts[1])
        assert torch.equal(a.counts, b.counts) and int(a.status[0]) == 0 and int(b.status[0]) == 0 and n > 0
        assert torch.equal(a.crd1[:n], b.crd1[:n]) and torch.equal(a.val[:n], b.val[:n])


def _keys(rng, n, extent):
    """Exactly n distinct sorted numbers below `extent`, spread over it."""
    gap = extent // n
    return np.arange(n) * gap + rng.integers(0, gap, n)


SHORT, MIDDLE, LONG_F64 = 3 * 512 - 64 - 8, 9 * 504 - 8, 10 * 504 - 8       # entries of a partition, less one an operand


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("fmt,line", [("vector", 2 * SHORT), ("csr", 2 * SHORT), ("csr few", 4 * SHORT), ("dcsr", 4 * SHORT * 5 / 6),
                                      ("coo", 4 * SHORT * 5 / 6), ("csf3", 4 * SHORT * 5 / 6)] +
                         [(f, 4 * MIDDLE) for f in ("vector", "csr", "dcsr", "coo", "csf3")] +
                         [(f, 4 * LONG_F64) for f in ("vector", "csr", "dcsr", "coo", "csf3")] + [("csr", 2 * MIDDLE), ("dcsr", 2 * MIDDLE)])
def test_merge_at_the_lines_between_lengths_of_partitions(fmt, line, dtype):
    """The last call with short, middle or (doubles) long partitions and the first without, every format, two or three
    operands, against the oracle."""
    if line == 4 * LONG_F64 and dtype == np.float32:
        line = 2 * (11 * 504 - 8)                           # (floats: two long ones a compute unit)
    rng = np.random.default_rng(int(line))
    for over in (0, 1):
        total = int(UNITS * line) + over
        k = 2 + over
        sizes = [total // k + (t < total % k) for t in range(k)]
        n_rows = {"csr": 4096, "csr few": 400_000, "dcsr": 60_000, "coo": 60_000}.get(fmt, 0)
        cells = {"vector": 1 << 30, "csf3": 60 * 256 * 4096}.get(fmt, n_rows << 16)
        keys = [_keys(rng, n, cells) for n in sizes]
        keys[1][::5] = keys[0][:len(keys[1][::5])]          # (some coordinates in two operands)
        keys[1] = np.unique(keys[1])
        if len(keys[1]) < sizes[1]:
            keys[1] = np.union1d(keys[1], np.setdiff1d(_keys(rng, 2 * sizes[1], cells), keys[1])[:sizes[1] - len(keys[1])])
        assert sum(len(x) for x in keys) == total
        vals = [rng.uniform(-1, 1, len(x)).astype(dtype) for x in keys]
        tag = f"line {line} {over}"
        if fmt == "vector":
            add.check_vec([x.astype(np.int32) for x in keys], vals, 1 << 30, 0, tag)
        elif fmt == "csf3":
            shape = (60, 256, 4096)
            csf3._check([csf3._tensor(np.stack(np.unravel_index(x, shape), 1), v) for x, v in zip(keys, vals)], shape, 0, tag)
        else:
            shape = (n_rows, 1 << 16)
            cs = [np.stack([x >> 16, x & 0xffff], 1) for x in keys]
            if fmt == "coo":
                coo._check(nb.nacho_spadd_k, oracle.spadd_coo, cs, vals, shape, 0, tag)
            else:
                (add.check_dcsr if fmt == "dcsr" else add.check_csr)(list(zip(cs, vals)), shape, 0, tag)


def _banded(rng, n_rows, n_cols, dense, sparse):
    """Many entries in a band of a few rows and a few in rows far apart: partitions of the latter span more rows than the
    row field of their keys holds."""
    top = rng.integers(0, 60, dense) * n_cols + rng.integers(0, n_cols, dense)
    rest = rng.integers(60, n_rows, sparse) * n_cols + rng.integers(0, n_cols, sparse)
    return np.unique(np.concatenate([top, rest]))


@pytest.mark.parametrize("k,total,dtype", [(2, 1_100_000, np.float32), (3, 1_100_000, np.float64),
                                           (2, 3_300_000, np.float64), (3, 3_300_000, np.float32),
                                           (2, 5_600_000, np.float32), (3, 5_600_000, np.float64)])
def test_merge_in_bands(k, total, dtype):
    """Rows past the row field (12 bits beside 2^20 columns): the partition is merged by searches; short partitions,
    middle and long ones."""
    rng = np.random.default_rng(41)
    shape = (1 << 19, 1 << 20)
    keys = [_banded(rng, *shape, int(total / (k + 0.33)), 9000) for _ in range(k)]
    keys[1] = np.unique(np.concatenate([keys[1], keys[0][::3]]))
    cs = [np.stack([x // shape[1], x % shape[1]], 1) for x in keys]
    mats = [(c, rng.uniform(-1, 1, len(c)).astype(dtype)) for c in cs]
    vals = [v for _, v in mats]
    add.check_dcsr(mats, shape, 0, "bands")
    add.check_csr(mats, shape, 0, "bands")
    coo._check(nb.nacho_spadd_k, oracle.spadd_coo, cs, vals, shape, 0, "add bands")
    coo._check(nb.nacho_spmul_k, oracle.spmul_coo, cs, vals, shape, 0, "mul bands")
    prods = []
    for c, v in mats:
        pos, crd = to_csr(c, shape[0])
        prods.append({"pos": pos, "crd": crd, "val": v})
    mul.check_csr(prods, shape, 0, "bands")


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("draws", [600_000, 1_500_000, 3_200_000])
def test_merge_tensors_in_bands(dtype, draws):
    """Slices past the row field of a tensor's keys (16 bits hold slice and fibre): short, middle and long partitions."""
    rng = np.random.default_rng(51)
    shape = (100_000, 64, 256)
    tens = []
    for _ in range(2):
        top = rng.integers(0, 400, draws) * (64 * 256) + rng.integers(0, 64 * 256, draws)
        rest = rng.integers(400, shape[0], 4000) * (64 * 256) + rng.integers(0, 64 * 256, 4000)
        lin = np.unique(np.concatenate([top, rest]))
        c = np.stack(np.unravel_index(lin, shape), axis=1)
        tens.append(csf3._tensor(c, rng.uniform(-1, 1, len(c)).astype(dtype)))
    csf3._check(tens, shape, 0, "bands")


@pytest.mark.parametrize("k,dtype", [(2, np.float32), (3, np.float64)])
def test_merge_few_rows_per_key(k, dtype):
    """Eight bits of row field beside 2^24 columns, thousands of rows in the first partitions; and a result that does not
    fit: what is written is the start of the whole result, what lies behind it stays."""
    rng = np.random.default_rng(61)
    shape = (65_000, 1 << 24)
    keys = []
    for _ in range(k):
        top = rng.integers(0, 60_000, 2500) * shape[1] + rng.integers(0, shape[1], 2500)
        rest = rng.integers(60_000, shape[0], 6_200_000 // k) * shape[1] + rng.integers(0, shape[1], 6_200_000 // k)
        keys.append(np.unique(np.concatenate([top, rest])))
    keys[1] = np.unique(np.concatenate([keys[1], keys[0][:3000:2]]))
    cs = [np.stack([x // shape[1], x % shape[1]], 1) for x in keys]
    mats = [(c, rng.uniform(-1, 1, len(c)).astype(dtype)) for c in cs]
    add.check_dcsr(mats, shape, 0, "few rows per key")
    ds = [mul_dcsr._mat(c, v) for c, v in mats]
    ops = [nb.dcsr(dev(m["pos0"]), dev(m["crd0"]), dev(m["pos1"]), dev(m["crd1"]), *shape, dev(m["val"])) for m in ds]
    total = sum(len(c) for c in cs)
    dt = torch.float32 if dtype == np.float32 else torch.float64
    whole = nb.nacho_spadd_k(ops, nb.SparseOut("dcsr", total, total, dt, "cuda"))
    for cap_rows, cap_nnz in ((total, 2999), (1777, total)):
        part_of = nb.SparseOut("dcsr", total, total, dt, "cuda")
        part_of.c.cap_rows, part_of.c.cap_nnz = cap_rows, cap_nnz
        for a in (part_of.crd0, part_of.pos1, part_of.crd1, part_of.val):
            a.fill_(-7)
        nb.nacho_spadd_k(ops, part_of)
        assert int(part_of.status[0]) == -4 and torch.equal(part_of.counts, whole.counts)
        rows, nnz = min(cap_rows, int(whole.counts[0])), min(cap_nnz, int(whole.counts[1]))
        for name, n in (("crd0", rows), ("pos1", rows), ("crd1", nnz), ("val", nnz)):
            got, ref = getattr(part_of, name), getattr(whole, name)
            assert torch.equal(got[:n], ref[:n]), name
            behind = n + (1 if name == "pos1" else 0)
            assert bool((got[behind:] == -7).all()), name


def _triples(rng, shape, n):
    c = np.stack([rng.integers(0, e, n) for e in shape], 1)
    return np.unique(c, axis=0)


@pytest.mark.parametrize("k,dtype", [(2, np.float64), (3, np.float32), (5, np.float32)])
def test_merge_tensors_wide(k, dtype):
    """64-bit keys: a second mode of 2^24 (any slice fits), modes with which 20, 17 and 2 bits are left for the slice, and
    slices, fibres and entries that two operands share."""
    rng = np.random.default_rng(71)
    top = (1 << 31) - 1
    for shape in ((1_000_000, 1 << 24, 16), (top, 1 << 24, 1 << 20), (top, top, 300), (top, top, top)):
        tens, first = [], None
        for t in range(k):
            c = _triples(rng, shape, 40_000 // k)
            if t == 0:
                first = c
            else:
                same = first[rng.choice(len(first), 3000, replace=False)]
                fibre, piece = same.copy(), same.copy()
                fibre[:, 2] = rng.integers(0, shape[2], len(same))
                piece[:, 1] = rng.integers(0, shape[1], len(same))
                c = np.unique(np.concatenate([c, same[:1500], fibre, piece]), axis=0)
            tens.append(csf3._tensor(c, rng.uniform(-1, 1, len(c)).astype(dtype)))
        for P in (0, 1, 37):
            csf3._check(tens, shape, P, "wide")


@pytest.mark.parametrize("k,dtype", [(2, np.float32), (2, np.float64), (3, np.float64)])
def test_product_rows_past_the_key(k, dtype):
    """Remapped operands: eight bits of row field beside 2^24 columns, thousands of common rows of one or two entries."""
    rng = np.random.default_rng(81)
    shape = (1 << 20, 1 << 24)
    thin = np.sort(rng.choice(np.arange(100, shape[0]), 4000, replace=False))
    shared = np.unique(thin * shape[1] + rng.integers(0, shape[1], len(thin)))
    wide = np.unique(rng.integers(0, 60, 30_000) * shape[1] + rng.integers(0, shape[1], 30_000))
    mats = []
    for _ in range(k):
        own = thin[rng.choice(len(thin), 2500, replace=False)] * shape[1] + rng.integers(0, shape[1], 2500)
        more = rng.integers(0, 60, 400_000) * shape[1] + rng.integers(0, shape[1], 400_000)
        keys = np.unique(np.concatenate([shared, own, wide, more]))
        c = np.stack([keys // shape[1], keys % shape[1]], 1)
        mats.append(mul_dcsr._mat(c, rng.uniform(0.5, 1, len(c)).astype(dtype)))
    mul_dcsr.check(mats, shape, 0, "rows past the key")


@pytest.mark.parametrize("k", [2, 5, 8])
@pytest.mark.parametrize("gap", [65533, 65534, 65535, 65536])
def test_merge_rows_at_the_limit_of_the_key(gap, k):
    """16 bits of row field beside 16 of column: the first partition holds two rows just within it, or just past it."""
    rng = np.random.default_rng(gap + k)
    shape = (200_000, 1 << 16)
    row = lambda r, n: r * shape[1] + rng.choice(shape[1], n, replace=False)
    both = np.concatenate([row(0, 100), row(gap, 400)])
    cs, vals = [], []
    for _ in range(k):
        keys = [both, row(0, 1000 // k), row(gap, 4000 // k)] + [row(199_000 + i, 30_000 // k) for i in range(2)]
        keys = np.unique(np.concatenate(keys))
        cs.append(np.stack([keys // shape[1], keys % shape[1]], 1))
        vals.append(rng.uniform(-1, 1, len(keys)).astype(np.float32))
    mats = list(zip(cs, vals))
    add.check_dcsr(mats, shape, 0, "limit")
    add.check_csr(mats, shape, 0, "limit")
    coo._check(nb.nacho_spadd_k, oracle.spadd_coo, cs, vals, shape, 0, "add limit")
    coo._check(nb.nacho_spmul_k, oracle.spmul_coo, cs, vals, shape, 0, "mul limit")
    mul.check_csr([dict(zip(("pos", "crd"), to_csr(c, shape[0])), val=v) for c, v in mats], shape, 0, "limit")


@pytest.mark.parametrize("k", [2, 3, 8])
@pytest.mark.parametrize("shape,gap", [((100_000, 64, 256), g) for g in (1021, 1022, 1023, 1024)] +
                         [((1 << 25, 1 << 24, 16), g) for g in (16_776_958, 16_776_959, 16_776_960, 16_777_216)])
def test_merge_slices_at_the_limit_of_the_key(shape, gap, k):
    """The same for the slices of tensors: ten bits beside six of the fibre (32-bit keys), 24 beside 24 (64-bit keys)."""
    rng = np.random.default_rng(gap + k)

    def slice_(i, n):
        c = np.stack([np.full(n, i), rng.integers(0, shape[1], n), rng.integers(0, shape[2], n)], 1)
        c[::3, 1] = shape[1] - 1
        return c

    both = np.concatenate([slice_(0, 100), slice_(gap, 400)])
    tens = []
    for _ in range(k):
        c = [both, slice_(0, 1000 // k), slice_(gap, 4000 // k)] + [slice_(shape[0] - 2 - i, 60_000 // k) for i in range(2)]
        c = np.unique(np.concatenate(c), axis=0)
        tens.append(csf3._tensor(c, rng.uniform(-1, 1, len(c)).astype(np.float32)))
    csf3._check(tens, shape, 0, "limit")


@pytest.mark.parametrize("k,dtype", [(2, np.float32), (3, np.float64), (8, np.float32)])
def test_merge_far_rows_beside_long_ones(k, dtype):
    """Eight bits of row field beside 2^24 columns; in one partition rows of one entry and rows of hundreds, which some
    or all of the operands store, with entries that some or all of them share."""
    rng = np.random.default_rng(91 + k)
    shape = (60_000, 1 << 24)
    long_rows = np.repeat(np.arange(40, 5000, 700), 300)
    common = np.unique(np.concatenate([long_rows * shape[1] + rng.integers(0, shape[1], len(long_rows)),
                                       rng.integers(0, 5000, 300) * shape[1] + rng.integers(0, 9, 300)]))
    cs, vals = [], []
    for t in range(k):
        own = np.repeat(np.arange(40 + 700 * (t % 3), 5000, 1400), 200)
        keys = np.unique(np.concatenate([common if t < 2 else common[rng.random(len(common)) < 0.7],
                                         own * shape[1] + rng.integers(0, shape[1], len(own)),
                                         rng.integers(0, 5000, 500) * shape[1] + rng.integers(0, 9, 500),
                                         59_990 * shape[1] + rng.integers(0, 10 * shape[1], 6_200_000 // k)]))
        cs.append(np.stack([keys // shape[1], keys % shape[1]], 1))
        vals.append(rng.uniform(-1, 1, len(keys)).astype(dtype))
    mats = list(zip(cs, vals))
    add.check_dcsr(mats, shape, 0, "far and long")
    add.check_csr(mats, shape, 0, "far and long")
    coo._check(nb.nacho_spadd_k, oracle.spadd_coo, cs, vals, shape, 0, "add far and long")
    coo._check(nb.nacho_spmul_k, oracle.spmul_coo, cs, vals, shape, 0, "mul far and long")
    mul_dcsr.check([mul_dcsr._mat(c, v) for c, v in mats], shape, 0, "far and long")


# ---- recursive partitioning -----------------------------------------------------
@pytest.mark.parametrize("rows", [511, 512, 513, 2047, 2048, 2049, 40_000, 140_000])
def test_product_row_loop(rows):
    """Row-loop partitions of 1024 coordinates and result tiles of 2048 rows, one more and one less; more workgroups
    than the 64 words a look-back step reads."""
    rng = np.random.default_rng(rows)
    shape = (3 * rows, 50)
    mats = []
    common = np.sort(rng.choice(shape[0], rows, replace=False))
    for t in range(2):
        own = rng.choice(shape[0], rows // 8, replace=False) if t and rows > 3000 else common[:0]
        r = np.unique(np.concatenate([common, own]))
        keys = np.unique(np.concatenate([r * 50 + rng.integers(0, 4, len(r)), r * 50 + rng.integers(0, 50, len(r))]))
        c = np.stack([keys // 50, keys % 50], 1)
        mats.append(mul_dcsr._mat(c, rng.uniform(0.5, 1, len(c)).astype(np.float32)))
    mul_dcsr.check(mats, shape, 0, "row loop")


@pytest.mark.parametrize("need,partitions", [(945, 945), (946, 1024), (1025, 1025), (1890, 1890), (1891, 2048), (2049, 2049)])
def test_merge_whole_rounds(need, partitions):
    """Partitions are rounded up to a whole number of rounds of workgroups where that adds a twelfth at most; the sum is
    that of the same call in other partitions, bit for bit."""
    capacity = 11 * 504 - 2                             # 11 places for each of 504 threads; shares differ by k at most
    total = need * capacity
    gen = torch.Generator(device="cuda").manual_seed(need)
    ops = []
    for n in (total - total // 3, total // 3):
        step = torch.randint(1, 90, (n,), device="cuda", generator=gen)
        keys = torch.cumsum(step, 0).to(torch.int32)
        ops.append(nb.vector(keys, (1 << 30) + 7, torch.rand(n, device="cuda", generator=gen)))
    print(f"whole rounds {need}", flush=True)
    if nb.num_partitions(nb.OP_SPADD, ops, nb.F32, 0, 1) != need:
        pytest.fail("the capacity of a partition has changed")
    assert nb.num_partitions(nb.OP_SPADD, ops, nb.F32) == partitions
    a, b = (nb.nacho_spadd_k(ops, nb.SparseOut("vector", 0, total, torch.float32, "cuda"), P=P) for P in (0, 2500))
    n = int(a.counts[1])
    assert torch.equal(a.counts, b.counts) and int(a.status[0]) == 0 and int(b.status[0]) == 0
    assert torch.equal(a.crd1[:n], b.crd1[:n]) and torch.equal(a.val[:n], b.val[:n])


def test_positions_up_to_the_last_one():
    """2^31 - 1 stored non-zeros, the most a call takes: positions of the last partitions and ends of the last rows lie
    less than a partition below 2^31.  Every sum is a whole number below 2^24: exact in any order."""
    rows, cols = 2048, 1 << 20
    nnz = rows * cols - 1
    pos = torch.arange(rows + 1, dtype=torch.int64, device="cuda").mul_(cols).clamp_(max=nnz).to(torch.int32)
    crd = torch.arange(cols, dtype=torch.int32, device="cuda").repeat(rows)[:nnz]
    op = nb.csr(pos, crd, rows, cols, torch.ones(nnz, dtype=torch.float32, device="cuda"))
    j = torch.arange(cols, device="cuda")
    for n in (0, 4):                                       # SpMV, SpMM
        B = ((j[:, None] + torch.arange(max(n, 1), device="cuda")) % 7).to(torch.float32)
        want = B.double().sum(0).expand(rows, -1).clone()
        want[-1] -= B[-1].double()                         # (the last row ends one column early)
        print(f"positions to the last one n={n}", flush=True)
        got = nb.nacho_spmm(op, B) if n else nb.nacho_spmv(op, B[:, 0].contiguous())[:, None]
        assert torch.equal(got.double(), want)


def test_the_stream_of_a_call_is_torchs_current_one():
    """The private getter and the public call it stands for name the same stream, on torch's default stream and on others."""
    for stream in (torch.cuda.default_stream(), torch.cuda.Stream(), torch.cuda.Stream()):
        with torch.cuda.stream(stream):
            assert nb._stream() == nb._public_stream() == stream.cuda_stream


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("shares", [(0.5, 0.5), (1.0, 0.0), (0.999, 0.001), (0.6, 0.3, 0.1), (0.5, 0.5, 0.0)])
def test_sums_whose_values_are_asked_for_ahead(shares, dtype):
    """Two and three tensors and coordinate lists just under and over the entries from which a partition asks for the lines of its
    values beside its merge: operands of equal length, next to nothing, none at all, and lines that two partitions share."""
    rng = np.random.default_rng(len(shares))
    shape = (300, 301, 4001)
    for total in (3_199_990, 3_200_011):
        keys = [np.unique(rng.integers(0, shape[0] * shape[1] * shape[2], int(total * s * 1.02) + 2, dtype=np.int64)) for s in shares]
        keys = [k[:int(round(total * s))] for k, s in zip(keys, shares)]
        vals = [rng.uniform(-1, 1, len(k)).astype(dtype) for k in keys]
        csf3._check([csf3._tensor(np.stack(np.unravel_index(k, shape), 1), v) for k, v in zip(keys, vals)], shape, 0, "values ahead")
        flat = (shape[0] * shape[1], shape[2])
        coo._check(nb.nacho_spadd_k, oracle.spadd_coo, [np.stack([k // flat[1], k % flat[1]], 1) for k in keys], vals, flat, 0, "values ahead")


@pytest.mark.parametrize("dtype,shares,total", [(d, s, t) for d in DTYPES for s in [(0.5, 0.5), (1.0, 0.0), (0.6, 0.3, 0.1), (0.3, 0.3, 0.3, 0.1)]
                                                for t in (1_249_280, 1_249_281)] +
                         [(np.float32, (0.4, 0.35, 0.25), t) for t in (14_000_000, 14_000_001)])
def test_lists_whose_values_are_asked_for_ahead(shares, total, dtype):
    """Two and three coordinate lists on both sides of the entries from which a partition asks for the lines of its values beside its
    merge, three lists on both sides of those up to which it does, and four, which never do."""
    rng = np.random.default_rng(len(shares))
    shape = (90_000, 40_001)
    counts = [int(total * s) for s in shares[:-1]]
    counts.append(total - sum(counts))
    keys = [np.sort(rng.permutation(np.unique(rng.integers(0, shape[0] * shape[1], n + n // 10 + 2, dtype=np.int64)))[:n]) for n in counts]
    assert sum(len(k) for k in keys) == total
    coo._check(nb.nacho_spadd_k, oracle.spadd_coo, [np.stack([k // shape[1], k % shape[1]], 1) for k in keys],
               [rng.uniform(-1, 1, len(k)).astype(dtype) for k in keys], shape, 0, "lists ahead")


# (non-zeros and rows on either side of the calls that do without a partition kernel, and the columns on either side of those)
WHOLE_LINES = [(np.float64, 524_289, 50_000, 524_288), (np.float64, 2_097_152, 200_000, 524_288),
               (np.float64, 2_097_153, 200_000, 327_680), (np.float64, 5_242_880, 400_000, 327_680),
               (np.float64, 5_242_881, 400_000, 327_680),
               (np.float32, 1_048_577, 100_000, 1_048_576), (np.float32, 2_097_152, 131_073, 1_048_576),
               (np.float32, 2_097_153, 131_072, 1_048_576), (np.float32, 2_097_153, 131_073, 1_048_576),
               (np.float32, 5_242_880, 131_072, 1_048_576), (np.float32, 5_242_881, 131_072, 1_048_576),
               (np.float32, 1_400_000, 20_000, 1_048_576), (np.float32, 4_194_305, 60_000, 1_048_576),
               (np.float32, 8_388_608, 131_072, 1_048_576), (np.float32, 8_388_609, 131_072, 1_048_576)]


@pytest.mark.parametrize("dtype,nnz,n_rows,n_cols", WHOLE_LINES)
def test_spmv_with_and_without_a_partition_kernel(dtype, nnz, n_rows, n_cols):
    """The same matrix with a column more, whose x is past what a call without a partition kernel may have: the same bits, and the
    oracle's values.  Rows of all lengths, empty ones, one that spans many partitions."""
    rng = np.random.default_rng(nnz % 1009)
    stored = np.union1d(np.flatnonzero(rng.random(n_rows) < 0.8), [n_rows // 3, n_rows - 1])
    lens = np.zeros(n_rows, np.int64)
    lens[stored] = rng.integers(0, max(1, nnz // (2 * n_rows)) + 1, len(stored))
    lens[n_rows // 3] = min(n_cols, nnz // 5)
    more, rest = divmod(nnz - int(lens.sum()), len(stored))
    lens[stored] += more
    lens[stored[:rest]] += 1
    lens = np.minimum(lens, n_cols)
    lens[-1] += nnz - int(lens.sum())
    pos = np.zeros(n_rows + 1, np.int32)
    pos[1:] = np.cumsum(lens)
    at = np.arange(nnz) - np.repeat(pos[:-1].astype(np.int64), lens)
    crd = (at * n_cols // np.repeat(np.maximum(lens, 1), lens)).astype(np.int32)
    A = {"n_rows": n_rows, "n_cols": n_cols, "pos": pos, "crd": crd, "val": rng.uniform(-1, 1, nnz).astype(dtype)}
    x = rng.uniform(-1, 1, n_cols).astype(dtype)
    y = spmv._check(A, x, 0, "without")
    wider = spmv._check(dict(A, n_cols=n_cols + 1), np.append(x, dtype(1)), 0, "with")
    assert np.array_equal(y.view(np.uint8), wider.view(np.uint8))


# entries of the operands: the last one has no partner in the merge's first round (five: the fifth), or the one before it has none because
# an operand is empty; a full short partition (1472 entries, less one an operand) and shares of more
LONE = [(734, 734, 1), (1, 1, 1467), (1, 734, 734), (700, 0, 769), (0, 1, 1468), (5, 0, 0, 1463), (3, 700, 0, 765),
        (366, 366, 366, 368, 1), (1, 1, 1, 1, 1463), (500, 0, 0, 0, 967), (300, 0, 400, 0, 767), (200, 200, 200, 200, 200, 200, 265)]


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("scale", [1, 2047, 5000])         # one short partition; middle ones; long ones (of doubles: middle again)
def test_runs_without_a_partner(scale, dtype):
    """Sums and products of three to seven operands, vectors and coordinate lists (one short partition of these with 64-bit keys too);
    operands share entries."""
    rng = np.random.default_rng(scale)
    for counts in LONE if scale == 1 else LONE[:2] + LONE[7:9]:
        total = scale * sum(counts)
        extent = 4 * total
        pool = rng.permutation(extent).astype(np.int32)
        vs = [np.sort(pool[:scale * n] if t % 2 == 0 else pool[scale * n // 2:scale * n // 2 + scale * n]) for t, n in enumerate(counts)]
        vals = [rng.uniform(-1, 1, len(v)).astype(dtype) for v in vs]
        add.check_vec(vs, vals, extent, 0, "lone run")
        mul.check_vec(vs, vals, extent, 0, "lone run")
        far = (2**31 - 1) // extent
        layouts = [((extent // 1000 + 1, 1000), lambda v: [v // 1000, v % 1000])]
        if scale == 1:
            layouts.append(((2**31 - 1, 2**31 - 1), lambda v: [v * far, v % 1000 * far]))
        for shape, place in layouts:
            lists = [np.stack(place(v.astype(np.int64)), 1) for v in vs]
            for fn, ref in ((nb.nacho_spadd_k, oracle.spadd_coo), (nb.nacho_spmul_k, oracle.spmul_coo)):
                coo._check(fn, ref, lists, vals, shape, 0, "lone run")
