"""GPU parity: nacho_spadd_fused (sparse vectors; the workgroups of the merge kernel search their own
boundaries, no partition kernel) against the oracle's k-finger union merge, and its partition table
against the oracle's Algorithm 1 (Section 3.2) on the equal-share queries.  Index arrays bit-exact,
values within 1e-5 (fp32) / 1e-12 (fp64)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2604_17198_amd import binding as nb
from paper_2604_17198_amd import workloads
from gpu_util import dev, vector_operand
from util import tol_ok

pytestmark = pytest.mark.gpu

TOL = {np.float32: 1e-5, np.float64: 1e-12}


def _check(vs, vals, extent, P, tag):
    dtype = vals[0].dtype.type
    ops = [nb.vector(dev(i), extent, dev(v)) for i, v in zip(vs, vals)]
    o = [oracle.vector(i, extent) for i in vs]
    total = sum(len(i) for i in vs)
    print(f"spadd fused {tag} k={len(vs)} sizes={[len(v) for v in vs]} P={P}", flush=True)
    dt = nb.dtype_code(dev(vals[0]).dtype)
    ws = torch.empty(nb.workspace_bytes(nb.OP_SPADD, ops, dt, 0, P), dtype=torch.uint8, device="cuda")
    ws.fill_(0xA5)                                     # nothing of the table is there before the call
    out = nb.SparseOut("vector", 0, total, dev(vals[0]).dtype, "cuda")
    out.status.fill_(77)
    nb.nacho_spadd_fused(ops, out, P=P, ws=ws)
    torch.cuda.synchronize()
    nnz = int(out.counts.cpu().numpy()[1])
    status = int(out.status.cpu().numpy()[0])
    ri, rv, ra = oracle.spadd_vec(vs, vals)
    assert status == 0 and nnz == ri.shape[0], (tag, status, nnz, ri.shape[0])
    assert np.array_equal(out.crd1.cpu().numpy()[:nnz], ri), tag
    assert out.pos1.cpu().numpy().tolist() == [0, nnz]
    ok = tol_ok(out.val.cpu().numpy()[:nnz], rv, ra, TOL[dtype])
    assert ok.all(), (tag, int((~ok).sum()))
    # the table the workgroups left behind is Algorithm 1's
    t = nb.workspace_parts(nb.OP_SPADD, ops, dt, ws, 0, P)
    ref = oracle.partition(o, t["P"])
    got = {name: t[name].cpu().numpy() for name in ("coord", "posn", "cost")}
    assert np.array_equal(got["cost"], ref["cost"]), tag
    assert np.array_equal(got["posn"].astype(np.int64), ref["posn"]), tag
    assert np.array_equal(got["coord"].astype(np.int64), ref["coord"][:, :got["coord"].shape[1]]), tag


@pytest.mark.parametrize("k", [1, 2, 3, 4, 5, 8])
@pytest.mark.parametrize("dtype", [np.float32, np.float64])
def test_vectors_random(k, dtype):
    rng = np.random.default_rng(700 + k)
    for trial in range(4):
        extent = int(rng.choice([50, 5000, 10**6, 2**30]))
        vs, vals = [], []
        for t in range(k):
            n = int(rng.integers(0, min(extent, 20000) + 1))
            idx = np.unique(rng.integers(0, extent, n)).astype(np.int32)
            if trial == 1 and t > 0:
                idx = vs[0].copy()                       # all coordinates tied
            if trial == 2 and t == 1:
                idx = np.zeros(0, np.int32)              # an empty operand
            vs.append(idx)
            vals.append(rng.uniform(-1, 1, idx.shape[0]).astype(dtype))
        for P in (0, 1, 13, 500):
            _check(vs, vals, extent, P, f"random{trial}")


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("k", [2, 3, 4, 5, 8])
def test_three_and_four_workgroups_on_a_compute_unit(k, dtype):
    """Up to three partitions a compute unit the kernel of long partitions runs, with more of them one held to the
    registers of four (from four or five operands on a kernel of its own, for middle partitions): both sides of
    the line, middle partitions as full as they get, and calls past a round, where doubles have middle ones again."""
    units = torch.cuda.get_device_properties(0).multi_processor_count
    rng = np.random.default_rng(750 + k)

    def vectors(total):
        vs = [np.unique(rng.integers(0, 2**30, total // k)).astype(np.int32) for _ in range(k)]
        vs[-1] = np.unique(np.concatenate([vs[-1][::2], vs[0][:len(vs[-1]) // 2]]))       # (some coordinates in two)
        return vs, [rng.uniform(-1, 1, len(v)).astype(dtype) for v in vs]

    vs, vals = vectors(units * 12_000)
    for P in (3 * units, 3 * units + 1):
        _check(vs, vals, 2**30, P, "line")
    for total, tag in ((units * 4 * 4528, "full"), (units * 4 * 5100, "past a round")):
        vs, vals = vectors(total)
        _check(vs, vals, 2**30, 0, tag)


def test_all_operands_empty():
    e = np.zeros(0, np.int32)
    _check([e, e], [e.astype(np.float32), e.astype(np.float32)], 100, 0, "empty")
    _check([e, e], [e.astype(np.float32), e.astype(np.float32)], 100, 7, "empty")


def test_config3_full_size_matches_the_unfused_call():
    cfg = workloads.config(3)
    ops = [vector_operand(v) for v in cfg["ops"]]
    total = sum(o.nnz for o in ops)
    a = nb.SparseOut("vector", 0, total, torch.float32, "cuda")
    b = nb.SparseOut("vector", 0, total, torch.float32, "cuda")
    wa = torch.empty(nb.workspace_bytes(nb.OP_SPADD, ops, nb.F32), dtype=torch.uint8, device="cuda")
    wb = torch.empty_like(wa)
    print(f"spadd fused C3 total={total}", flush=True)
    nb.nacho_spadd_k(ops, a, ws=wa)
    nb.nacho_spadd_fused(ops, b, ws=wb)
    torch.cuda.synchronize()
    assert int(b.status.cpu()[0]) == 0
    n = int(a.counts.cpu().numpy()[1])
    assert int(b.counts.cpu().numpy()[1]) == n
    assert torch.equal(a.crd1[:n], b.crd1[:n])
    assert torch.equal(a.val[:n], b.val[:n])            # same partitions, same order of additions
    ta = nb.workspace_parts(nb.OP_SPADD, ops, nb.F32, wa)
    tb = nb.workspace_parts(nb.OP_SPADD, ops, nb.F32, wb)
    for name in ("coord", "posn", "cost"):
        assert torch.equal(ta[name], tb[name]), name


def test_other_formats_are_refused():
    m = workloads.csr_powerlaw(50, 50, 300, 1.2, 20, 0.0, 3, np.float32)
    from gpu_util import csr_operand
    g = csr_operand(m)
    out = nb.SparseOut("csr", 0, 600, torch.float32, "cuda", n_rows=50)
    with pytest.raises(Exception):
        nb.nacho_spadd_fused([g, g], out)
