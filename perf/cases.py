"""What a program that uses this library has it do, as timed cases.

The listed cases span the calls users make: one SpMV inside an iterative solver (from 40 thousand to 50
million stored non-zeros), SpMM with a block of dense columns, k-way addition of sparse vectors, CSR, DCSR and
COO matrices and third-order CSF tensors, and element-wise products.  Sizes are those of the benchmark's
configurations, of the tests, and odd ones between them; `draw` spreads further cases over the same ranges.

Inputs are made on the GPU from a seed: row lengths follow the rank-frequency form of Zipf's law (a few rows
hold a large part of the entries, most hold a handful), columns are uniform inside a row and sorted, values are
uniform in [-1, 1).  A program keeps operands, result arrays and, where `kept` is set, the workspace from one
call to the next; where it is not, every call brings up its own workspace (and result, where the call makes one),
as a program without a loop around the call does.
"""
from __future__ import annotations

import math

import torch

from paper_2604_17198_amd import binding as nb

DEVICE = "cuda"


# --------------------------------------------------------------------------- #
# the cases
# --------------------------------------------------------------------------- #
def listed():
    return [
        # a small solver matrix: three short kernels, the call itself is what is waited for
        dict(name="spmv_small_f64", op="spmv", fmt="csr", dtype="f64", rows=4096, cols=4096, nnz=40_000,
             alpha=1.5, cap=0.9, empty=0.30, kept=True),
        # an ordinary single-precision SpMV on an odd, rectangular matrix, called without buffers in hand
        dict(name="spmv_mid_f32", op="spmv", fmt="csr", dtype="f32", rows=99_991, cols=120_011, nnz=5_000_000,
             alpha=1.3, cap=0.25, empty=0.0, kept=False),
        # the large power-law SpMV: 2M x 2M, 50M non-zeros
        dict(name="spmv_large_f64", op="spmv", fmt="csr", dtype="f64", rows=2_000_000, cols=2_000_000,
             nnz=50_000_000, alpha=1.3, cap=0.5, empty=0.30, kept=True),
        # SpMM with a few more right-hand sides than half a wavefront, double precision, ragged sizes
        dict(name="spmm_odd_f64", op="spmm", fmt="csr", dtype="f64", rows=65_537, cols=50_021, nnz=1_300_003,
             alpha=1.3, cap=0.25, empty=0.30, n=37, kept=False),
        # the large SpMM: 1M x 1M, 30M non-zeros, 64 feature columns
        dict(name="spmm_large_f32", op="spmm", fmt="csr", dtype="f32", rows=1_000_000, cols=1_000_000,
             nnz=30_000_000, alpha=1.3, cap=0.25, empty=0.0, n=64, kept=True),
        # two short sparse vectors: a sparse update inside a loop
        dict(name="spadd_vec2_small_f64", op="spadd", fmt="vector", dtype="f64", k=2, cols=1 << 20, nnz=20_001,
             ratio=0.5, share=0.2, kept=True),
        # three sparse vectors of very different lengths (10M, 1M, 100k)
        dict(name="spadd_vec3_large_f32", op="spadd", fmt="vector", dtype="f32", k=3, cols=1 << 30, nnz=10_000_000,
             ratio=0.1, share=0.2, kept=True),
        # three power-law CSR matrices summed in one call
        dict(name="spadd_csr3_f32", op="spadd", fmt="csr", dtype="f32", k=3, rows=100_000, cols=100_000,
             nnz=5_000_000, alpha=1.3, cap=0.25, empty=0.0, share=0.0, kept=True),
        # two hyper-sparse matrices (one row in ten stored, half of the rows in both), the largest sum
        dict(name="spadd_dcsr2_large_f32", op="spadd", fmt="dcsr", dtype="f32", k=2, rows=1_000_000, cols=1_000_000,
             nnz=20_000_000, alpha=1.4, cap=0.25, stored=0.10, share=0.0, kept=True),
        # coordinate lists in double precision, an assembly of two contributions
        dict(name="spadd_coo2_f64", op="spadd", fmt="coo", dtype="f64", k=2, rows=300_007, cols=250_003,
             nnz=2_500_000, alpha=1.3, cap=0.25, stored=0.5, share=0.2, kept=False),
        # third-order tensors of a few thousand coordinates per mode
        dict(name="spadd_csf2_f32", op="spadd", fmt="csf3", dtype="f32", k=2, rows=2000, cols=2000, depth=2000,
             nnz=8_000_000, share=0.2, kept=True),
        # element-wise product of the hyper-sparse matrices: an outer intersection
        dict(name="spmul_dcsr2_large_f32", op="spmul", fmt="dcsr", dtype="f32", k=2, rows=1_000_000, cols=1_000_000,
             nnz=20_000_000, alpha=1.4, cap=0.25, stored=0.10, share=0.2, kept=True),
    ]


def _spread(rng, lo, hi):
    """A whole number from [lo, hi], spread over its logarithm."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["spmv", "spmv", "spmm", "spadd", "spadd", "spadd", "spadd", "spmul"])
    c = dict(op=kind, dtype=rng.choice(["f32", "f64"]), kept=rng.random() < 0.7)
    if kind in ("spmv", "spmm"):
        c["fmt"] = "csr"
        c["nnz"] = _spread(rng, 20_000, 50_000_000 if kind == "spmv" else 10_000_000)
        c["rows"] = min(2_000_000, max(500, int(c["nnz"] / _spread(rng, 5, 100))))
        c["cols"] = max(500, int(c["rows"] * rng.uniform(0.5, 1.5)))
        c["alpha"] = round(rng.uniform(1.2, 1.5), 2)
        c["cap"] = rng.choice([0.25, 0.5, 0.9])
        c["empty"] = rng.choice([0.0, 0.3])
        if kind == "spmm":
            most = 30_000_000 * 64 // c["nnz"] // (2 if c["dtype"] == "f64" else 1)
            c["n"] = min(_spread(rng, 4, 200), max(4, most))
        return c
    c["fmt"] = rng.choice(["vector", "csr", "dcsr", "coo", "csf3"] if kind == "spadd" else
                          ["vector", "csr", "dcsr", "coo"])
    c["k"] = rng.choice([2, 2, 2, 3, 3, 4, 5, 8])
    c["share"] = rng.choice([0.0, 0.2])
    total = _spread(rng, 20_000, 20_000_000 if c["dtype"] == "f64" or c["k"] > 4 else 35_000_000)
    if c["fmt"] == "vector":
        c["ratio"] = rng.choice([0.1, 0.5, 1.0])           # every operand has this share of the one before it
        whole = sum(c["ratio"] ** t for t in range(c["k"]))
        c["nnz"] = max(1000, int(total / whole))
        c["cols"] = min((1 << 30) + 7, c["nnz"] * _spread(rng, 4, 1000))
        return c
    c["nnz"] = max(1000, total // c["k"])
    if c["fmt"] == "csf3":
        side = max(20, int((c["nnz"] * _spread(rng, 10, 2000)) ** (1.0 / 3.0)))
        c["rows"], c["cols"], c["depth"] = (max(20, int(side * rng.uniform(0.7, 1.4))) for _ in range(3))
        return c
    c["alpha"] = round(rng.uniform(1.2, 1.5), 2)
    c["cap"] = 0.25
    if c["fmt"] == "csr":
        c["rows"] = min(1_000_000, max(500, int(c["nnz"] / _spread(rng, 5, 100))))
        c["empty"] = rng.choice([0.0, 0.3])
    else:
        c["stored"] = rng.choice([0.1, 0.5])
        c["rows"] = min(1_000_000, max(500, int(c["nnz"] / c["stored"] / _spread(rng, 5, 200))))
    c["cols"] = max(500, int(c["rows"] * rng.uniform(0.5, 1.5)))
    return c


# --------------------------------------------------------------------------- #
# inputs
# --------------------------------------------------------------------------- #
class _Maker:
    """Seeded random arrays on the GPU."""

    def __init__(self, seed, dtype):
        self.gen = torch.Generator(device=DEVICE)
        self.gen.manual_seed(int(seed))
        self.dtype = dtype

    def values(self, *shape):
        return torch.rand(shape, dtype=self.dtype, device=DEVICE, generator=self.gen) * 2 - 1

    def below(self, n, count):
        return torch.randint(0, int(n), (int(count),), dtype=torch.int64, device=DEVICE, generator=self.gen)

    def some_of(self, a, count):
        """`count` of the elements of `a`, without replacement."""
        return a[torch.randperm(a.numel(), device=DEVICE, generator=self.gen)[:int(count)]]

    def at_most(self, a, count):
        """The sorted array `a`, cut down to `count` of its elements where it has more."""
        return a if a.numel() <= count else self.some_of(a, count).sort().values

    def distinct(self, extent, count):
        """About `count` distinct whole numbers below `extent`, at most that many, sorted (draws with
        repetition, so many that the distinct ones among them come to `count`)."""
        count = min(int(count), int(0.9 * extent))
        draws = int(round(-extent * math.log1p(-count / extent)))
        return self.at_most(torch.unique(self.below(extent, max(1, draws))), count)

    def row_lengths(self, n, nnz, alpha, cap):
        """Zipf's law by rank, each length in [1, cap], together about `nnz`; ranks meet rows at random."""
        w = torch.arange(1, n + 1, dtype=torch.float64, device=DEVICE) ** -alpha
        total = lambda s: float(torch.clamp(torch.floor(s * w), 1, cap).sum())
        lo, hi = 0.0, 1.0
        while total(hi) < nnz and hi < 1e18:
            hi *= 4.0
        for _ in range(40):
            mid = 0.5 * (lo + hi)
            lo, hi = (mid, hi) if total(mid) < nnz else (lo, mid)
        lengths = torch.clamp(torch.floor(hi * w), 1, cap)
        return lengths[torch.randperm(n, device=DEVICE, generator=self.gen)]

    def keys(self, rows, n_cols, nnz, alpha, cap):
        """row * n_cols + column of the entries of a power-law matrix with the given rows, sorted: about `nnz`
        of them, at most that many."""
        lengths = self.row_lengths(rows.numel(), nnz, alpha, max(1, int(cap * n_cols)))
        draws = torch.round(-n_cols * torch.log1p(-torch.clamp(lengths / n_cols, max=0.9))).to(torch.int64)
        row = torch.repeat_interleave(rows, draws)
        keys = torch.unique_consecutive(torch.sort(row * n_cols + self.below(n_cols, row.numel())).values)
        return self.at_most(keys, nnz)


def _i32(t):
    return t.to(torch.int32).contiguous()


def _starts(counts):
    pos = torch.zeros(counts.numel() + 1, dtype=torch.int64, device=DEVICE)
    torch.cumsum(counts, 0, out=pos[1:])
    return _i32(pos)


def _csr(m, keys, n_rows, n_cols):
    row = torch.div(keys, n_cols, rounding_mode="floor")
    pos = _starts(torch.bincount(row, minlength=n_rows))
    return nb.csr(pos, _i32(keys - row * n_cols), n_rows, n_cols, m.values(keys.numel()))


def _dcsr(m, keys, n_rows, n_cols):
    row = torch.div(keys, n_cols, rounding_mode="floor")
    stored, counts = torch.unique_consecutive(row, return_counts=True)
    pos0 = torch.tensor([0, stored.numel()], dtype=torch.int32, device=DEVICE)
    return nb.dcsr(pos0, _i32(stored), _starts(counts), _i32(keys - row * n_cols), n_rows, n_cols,
                   m.values(keys.numel()))


def _coo(m, keys, n_rows, n_cols):
    row = torch.div(keys, n_cols, rounding_mode="floor")
    return nb.coo(_i32(row), _i32(keys - row * n_cols), n_rows, n_cols, m.values(keys.numel()))


def _csf3(m, keys, shape):
    ij = torch.div(keys, shape[2], rounding_mode="floor")
    fibre, entries = torch.unique_consecutive(ij, return_counts=True)
    i = torch.div(fibre, shape[1], rounding_mode="floor")
    slices, fibres = torch.unique_consecutive(i, return_counts=True)
    pos0 = torch.tensor([0, slices.numel()], dtype=torch.int32, device=DEVICE)
    return nb.csf3(pos0, _i32(slices), _starts(fibres), _i32(fibre - i * shape[1]), _starts(entries),
                   _i32(keys - ij * shape[2]), shape, m.values(keys.numel()))


def _entries(c):
    """Stored entries of the k operands (of a vector sum every operand has `ratio` of the one before it)."""
    return [max(1, int(c["nnz"] * c.get("ratio", 1.0) ** t)) for t in range(c["k"])]


def _operand_keys(m, c):
    """The entries of the k operands of a sum or product as sorted numbers; a share of the later operands'
    entries is taken from the first one's."""
    def shared_with(first, own, count, ok=None):
        if count <= 0:
            return own
        pick = m.some_of(first, min(count, first.numel()))
        if ok is not None:
            pick = pick[ok(pick)]
        return torch.unique(torch.cat([own, pick]))

    out = []
    for t, n in enumerate(_entries(c)):
        ok = None
        n_shared = int(c["share"] * n) if t else 0
        if c["fmt"] == "vector":
            own = m.distinct(c["cols"], n - n_shared)
        elif c["fmt"] == "csf3":
            own = m.distinct(c["rows"] * c["cols"] * c["depth"], n - n_shared)
        else:
            if c["fmt"] == "csr":
                some = max(1, int(c["rows"] * (1.0 - c["empty"])))
                rows = m.some_of(torch.arange(c["rows"], device=DEVICE), some).sort().values
            else:
                some = max(1, int(c["rows"] * c["stored"]))
                if t == 0:
                    rows = first_rows = m.some_of(torch.arange(c["rows"], device=DEVICE), some).sort().values
                else:                                       # half of the stored rows are the first operand's
                    rest = torch.ones(c["rows"], dtype=torch.bool, device=DEVICE)
                    rest[first_rows] = False
                    fresh = m.some_of(torch.nonzero(rest).reshape(-1), some - some // 2)
                    rows = torch.cat([m.some_of(first_rows, some // 2), fresh]).sort().values
                    stored = torch.zeros(c["rows"], dtype=torch.bool, device=DEVICE)
                    stored[rows] = True
                    ok = lambda pick, stored=stored: stored[torch.div(pick, c["cols"], rounding_mode="floor")]
            own = m.keys(rows, c["cols"], n - n_shared, c["alpha"], c["cap"])
        out.append(own if t == 0 else shared_with(out[0], own, n_shared, ok))
    return out


def prepare(case, seed):
    c = case
    m = _Maker(seed, torch.float64 if c["dtype"] == "f64" else torch.float32)
    code = nb.F64 if c["dtype"] == "f64" else nb.F32
    state = {"op": c["op"], "ws": None}
    if c["op"] in ("spmv", "spmm"):
        some = max(1, int(c["rows"] * (1.0 - c["empty"])))
        rows = m.some_of(torch.arange(c["rows"], device=DEVICE), some).sort().values
        A = _csr(m, m.keys(rows, c["cols"], c["nnz"], c["alpha"], c["cap"]), c["rows"], c["cols"])
        n = c.get("n", 0)
        state["A"] = A
        state["x"] = m.values(c["cols"], n) if n else m.values(c["cols"])
        state["y"] = None
        if c["kept"]:
            state["y"] = torch.zeros((c["rows"], n) if n else c["rows"], dtype=m.dtype, device=DEVICE)
            size = nb.workspace_bytes(nb.OP_SPMM if n else nb.OP_SPMV, [A], code, n)
            state["ws"] = torch.empty(size, dtype=torch.uint8, device=DEVICE)
        return state
    ops = []
    for keys in _operand_keys(m, c):
        if c["fmt"] == "vector":
            ops.append(nb.vector(_i32(keys), c["cols"], m.values(keys.numel())))
        elif c["fmt"] == "csr":
            ops.append(_csr(m, keys, c["rows"], c["cols"]))
        elif c["fmt"] == "coo":
            ops.append(_coo(m, keys, c["rows"], c["cols"]))
        elif c["fmt"] == "dcsr":
            ops.append(_dcsr(m, keys, c["rows"], c["cols"]))
        else:
            ops.append(_csf3(m, keys, (c["rows"], c["cols"], c["depth"])))
    # capacities that always suffice: everything for a sum, the smallest operand for a product
    each = _entries(c)
    most = min if c["op"] == "spmul" else sum
    cap_rows = cap_fibres = 0
    if c["fmt"] == "dcsr":
        cap_rows = most([int(c["rows"] * c["stored"])] * c["k"])
    elif c["fmt"] == "csf3":
        cap_rows = c["rows"]
        cap_fibres = min(c["rows"] * c["cols"], sum(each))
    out = nb.SparseOut(c["fmt"], cap_rows, most(each), m.dtype, DEVICE, n_rows=c.get("rows", 0),
                       cap_fibres=cap_fibres)
    for a in (out.crd0, out.crd1, out.crd2, out.val):      # (what lies past the result stays zero)
        if a is not None:
            a.zero_()
    state["ops"], state["out"] = ops, out
    if c["kept"]:
        size = nb.workspace_bytes(nb.OP_SPMUL if c["op"] == "spmul" else nb.OP_SPADD, ops, code)
        state["ws"] = torch.empty(size, dtype=torch.uint8, device=DEVICE)
    return state


# --------------------------------------------------------------------------- #
# one call
# --------------------------------------------------------------------------- #
def run(state):
    if state["op"] == "spmv":
        return nb.nacho_spmv(state["A"], state["x"], state["y"], ws=state["ws"])
    if state["op"] == "spmm":
        return nb.nacho_spmm(state["A"], state["x"], state["y"], ws=state["ws"])
    call = nb.nacho_spmul_k if state["op"] == "spmul" else nb.nacho_spadd_k
    out = call(state["ops"], state["out"], ws=state["ws"])
    arrays = dict(pos0=out.pos0, crd0=out.crd0, pos1=out.pos1, crd1=out.crd1, pos2=out.pos2, crd2=out.crd2,
                  val=out.val, counts=out.counts, status=out.status)
    return {name: a for name, a in arrays.items() if a is not None}


def work(case):
    """Every operand array read once, every result array written once (nominal entry counts)."""
    c = case
    v = 8 if c["dtype"] == "f64" else 4
    if c["op"] in ("spmv", "spmm"):
        n = c.get("n", 1)
        size = c["nnz"] * (4 + v) + (c["rows"] + 1) * 4 + (c["cols"] + c["rows"]) * n * v
        return {"bytes": size, "flops": 2 * c["nnz"] * n}
    k = c["k"]
    each = _entries(c)
    common = c["share"]
    total = sum(each)
    if c["op"] == "spadd":
        result = total - int(common * sum(each[1:]))
    else:
        result = int(min(each) * common ** (k - 1))
    entry = (8 if c["fmt"] == "coo" else 4) + v
    read = total
    upper = 0
    if c["fmt"] == "csr":
        upper = (k + 1) * (c["rows"] + 1) * 4
    elif c["fmt"] == "dcsr":
        rows = int(c["rows"] * c["stored"])
        if c["op"] == "spmul":                              # rows that one operand lacks are not read below their coordinate
            read = total // 2 if k == 2 else total // k
            upper = k * rows * 8
        else:
            upper = k * rows * 8 + int(rows * (1 + 0.5 * (k - 1))) * 8
    elif c["fmt"] == "csf3":
        ij = c["rows"] * c["cols"]
        filled = lambda n: int(ij * -math.expm1(-n / ij))
        upper = (sum(filled(n) for n in each) + filled(result)) * 8 + (k + 1) * c["rows"] * 8
    return {"bytes": (read + result) * entry + upper, "flops": total}


def tolerance(case):
    """Sums in another order at the same precision; coordinates, positions, counts and status are exact."""
    return {"rel": 1e-12} if case["dtype"] == "f64" else {"rel": 1e-5}
