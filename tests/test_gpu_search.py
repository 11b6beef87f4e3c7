"""GPU parity of the boundary search where its expectations fail: operands that are spread nothing alike, windows of one
operand inside a gap of another, lengths on both sides of the lanes an operand gets (64 / k), heavy rows.  Every boundary
of a fine partition is compared with the oracle's Algorithm 1, bit-exact."""
import numpy as np
import pytest

import oracle
from paper_2604_17198_amd import binding as nb
from gpu_util import dev, parts_to_numpy
from util import to_csf3, to_csr, to_dcsr

pytestmark = pytest.mark.gpu

EXTENT = 1 << 24


def _spread(rng, kind, t, k):
    """The sorted distinct keys of operand t of k, below EXTENT."""
    n = int(rng.integers(200, 3000))
    if kind == "alike":
        x = rng.integers(0, EXTENT, n)
    elif kind == "apart":                              # one range behind the other
        x = t * (EXTENT // k) + rng.integers(0, EXTENT // k, n)
    elif kind == "inside":                             # every operand inside a gap of the one before
        x = np.concatenate([[0, EXTENT - 1 - t], EXTENT // 2 + rng.integers(0, EXTENT >> (2 + 2 * t), n)])
    elif kind == "bent":                               # density falls and rises by orders of magnitude
        x = (EXTENT - 1) * rng.random(n) ** (2 + 3 * t if t % 2 == 0 else 1 / (2 + 3 * t))
    elif kind == "steps":                              # powers of two, and runs without gaps
        x = np.concatenate([2 ** rng.integers(0, 24, 60) - 1, (EXTENT // (t + 2)) + np.arange(n)])
    else:                                              # "lanes": around the number of lanes an operand gets
        x = rng.integers(0, EXTENT, max(1, 64 // k + t - 2))
    return np.unique(np.asarray(x, dtype=np.int64).clip(0, EXTENT - 1))


def _operands(fmt, keys):
    rows, cols = 1 << 10, 1 << 14
    g, o = [], []
    for x in keys:
        c = np.stack([x // cols, x % cols], axis=1)
        if fmt == "vector":
            v = x.astype(np.int32)
            g.append(nb.vector(dev(v), EXTENT))
            o.append(oracle.vector(v, EXTENT))
        elif fmt == "csr":
            pos, crd = to_csr(c, rows)
            g.append(nb.csr(dev(pos), dev(crd), rows, cols))
            o.append(oracle.csr(pos, crd, rows, cols))
        elif fmt == "dcsr":
            a = to_dcsr(c)
            g.append(nb.dcsr(*[dev(y) for y in a], rows, cols))
            o.append(oracle.dcsr(*a, rows, cols))
        elif fmt == "coo":
            r, cc = c[:, 0].astype(np.int32), c[:, 1].astype(np.int32)
            g.append(nb.coo(dev(r), dev(cc), rows, cols))
            o.append(oracle.coo(r, cc, rows, cols))
        else:
            shape = (1 << 8, 1 << 8, 1 << 8)
            a = to_csf3(np.stack([x >> 16, x >> 8 & 255, x & 255], axis=1))
            g.append(nb.csf3(*[dev(y) for y in a], shape))
            o.append(oracle.Tensor([("compressed", shape[m], a[2 * m], a[2 * m + 1]) for m in range(3)]))
    return g, o


@pytest.mark.parametrize("kind", ["alike", "apart", "inside", "bent", "steps", "lanes"])
@pytest.mark.parametrize("fmt", ["vector", "csr", "dcsr", "coo", "csf3"])
def test_every_boundary(fmt, kind):
    for k in range(1, 9):
        rng = np.random.default_rng([k, len(fmt), len(kind), ord(kind[0])])
        keys = [_spread(rng, kind, t, k) for t in range(k)]
        if k > 4:
            keys[1] = keys[1][:0]                      # an operand without entries
        g, o = _operands(fmt, keys)
        total = sum(x.shape[0] for x in keys)
        for P in (3, 61, total + 3):
            print(f"partition {fmt} {kind} k={k} total={total} P={P}", flush=True)
            got, ref = parts_to_numpy(nb.nacho_partition(g, P)), oracle.partition(o, P)
            assert np.array_equal(got["cost"], ref["cost"]), (k, P)
            assert np.array_equal(got["coord"].astype(np.int64), ref["coord"][:, :got["coord"].shape[1]]), (k, P)
            assert np.array_equal(got["posn"].astype(np.int64), ref["posn"]), (k, P)


@pytest.mark.parametrize("fmt", ["vector", "csr", "dcsr", "coo", "csf3"])
def test_two_operands_around_the_lanes(fmt):
    """Every boundary of two operands as long as a wavefront has lanes, an entry or two fewer or more: all of it in one row
    (of one fibre), behind an empty row, the operands equal, apart, interleaved."""
    for n, m in ((1, 1), (61, 61), (62, 61), (62, 63), (63, 200), (64, 64), (126, 65), (1, 300)):
        for step, shift in ((1, 0), (1, 1), (2, 1), (1, n)):
            base = 3 << 14
            keys = [base + step * np.arange(n, dtype=np.int64), base + shift + step * np.arange(m, dtype=np.int64)]
            g, o = _operands(fmt, keys)
            P = n + m
            print(f"partition {fmt} {n} + {m} step {step} shift {shift}", flush=True)
            got, ref = parts_to_numpy(nb.nacho_partition(g, P)), oracle.partition(o, P)
            assert np.array_equal(got["cost"], ref["cost"])
            assert np.array_equal(got["coord"].astype(np.int64), ref["coord"][:, :got["coord"].shape[1]])
            assert np.array_equal(got["posn"].astype(np.int64), ref["posn"])


@pytest.mark.parametrize("k", [3, 8])
@pytest.mark.parametrize("fmt", ["vector", "csr", "dcsr", "coo", "csf3"])
def test_skewed_operands(fmt, k):
    """Hundreds of thousands of entries an operand, lengths and densities orders of magnitude apart."""
    rng = np.random.default_rng([k, len(fmt)])
    keys = []
    for t in range(k):
        n = [300_000, 700, 120_000, 500_000, 9, 250_000, 60_000, 400_000][t]
        x = rng.random(n) ** (1 + 4 * (t % 3) if t % 2 == 0 else 1 / (1 + 3 * t))
        if t == 3:
            x = 0.4 + x / 64                            # all of it in one place
        keys.append(np.unique((x * (EXTENT - 1)).astype(np.int64)))
    g, o = _operands(fmt, keys)
    for P in (1000, 1537):
        print(f"partition skewed {fmt} k={k} P={P}", flush=True)
        got, ref = parts_to_numpy(nb.nacho_partition(g, P)), oracle.partition(o, P)
        assert np.array_equal(got["cost"], ref["cost"])
        assert np.array_equal(got["coord"].astype(np.int64), ref["coord"][:, :got["coord"].shape[1]])
        assert np.array_equal(got["posn"].astype(np.int64), ref["posn"])


@pytest.mark.parametrize("sizes", [(40_000_000, 3_000_000, 100_000), (20_000_000,) + (1_000_000,) * 7])
def test_windows_past_single_precision(sizes):
    """Vectors of more than 2^24 entries, where the places of samples are further apart than floats tell."""
    extent, g, o = 2**31 - 1, [], []
    for t, n in enumerate(sizes):
        i = np.arange(n, dtype=np.int64)
        x = i + (i * i // n * 40 if t == 0 else np.where(i < n // 3, 0, extent // 5 * (1 + t % 4)))
        v = x.astype(np.int32)
        g.append(nb.vector(dev(v), extent))
        o.append(oracle.vector(v, extent))
    print(f"partition k={len(sizes)} of {sizes[0]}", flush=True)
    got, ref = parts_to_numpy(nb.nacho_partition(g, 700)), oracle.partition(o, 700)
    for name in ("cost", "posn"):
        assert np.array_equal(got[name].astype(np.int64), ref[name])
    assert np.array_equal(got["coord"][:, 0].astype(np.int64), ref["coord"][:, 0])
