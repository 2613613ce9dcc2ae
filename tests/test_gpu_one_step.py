"""Calls of one step, which make their tiles' records themselves, against calls
of several, which plan them: the same arithmetic, so the first of two recorded
steps and a recorded step alone agree bit for bit -- rows shorter than a window,
around one and two tiles, odd lengths, arrays off 16-byte alignment, meshes with
uniform runs, without, with a huge cell and with windows beyond the LDS, every
cumulative mode, FP32 and FP64.

Calls of an odd number of steps start from a copy of the state and end in place:
1, 3 and 5 in-place steps equal the recorded trajectory bit for bit, also on
per-row meshes, a schedule of the general kernel, limited steps and states whose
size is no multiple of 16 bytes.
"""
import numpy as np
import pytest
import torch

from paper_2305_05362_amd import _lib as R
from paper_2305_05362_amd import workloads as W

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")
SCANS = {torch.float32: [R.RAM_SCAN_F64, R.RAM_SCAN_F32_TWOSUM, R.RAM_SCAN_F32, R.RAM_SUM_DIRECT],
         torch.float64: [R.RAM_SCAN_F64, R.RAM_SUM_DIRECT]}


def dev(a, dtype=torch.float64, offset=0):
    a = torch.as_tensor(np.ascontiguousarray(a).reshape(-1), dtype=dtype)
    buf = torch.empty(a.numel() + offset, dtype=dtype, device=DEV)
    buf[offset:] = a.to(DEV)
    return buf[offset:]


def edges(kind, n):
    if kind == "uniform":
        return W.uniform_edges(n, 0.0, 1.0)
    if kind == "stretched":
        return W.stretched_edges(n, 6.0, np.random.default_rng(n))
    w = np.ones(n)
    if kind == "runs":                               # two uniform runs, a jump between them
        w[n // 3:2 * n // 3] = 0.1
    elif kind == "huge":
        w[n // 2] = 1.5 * n
    else:
        w[:4 * n // 5] = 0.02                        # windows beyond the LDS
    e = np.concatenate([[0.0], np.cumsum(w)]) / w.sum()
    e[-1] = 1.0
    return e


def inputs(n, kind, rows, with_dv, dtype, offset):
    rng = np.random.default_rng(n + rows)
    e = edges(kind, n)
    q = 1.0 + 0.2 * rng.standard_normal((rows, n))
    dv, dt = None, 1.0
    if with_dv:
        dv = rng.uniform(-1, 1, (rows, n))
        dt = W.residual_cfl_dt(e, dv, 0.4)
    v0 = rng.uniform(-0.7, 0.7, rows) / dt
    wl = W.Workload("one", rows, n, np.arange(rows + 1) * n, e, True, q, dv, v0, dt, 5, 1)
    return (R.Rows.from_workload(wl, DEV), dev(q, dtype, offset), dev(v0),
            None if dv is None else dev(dv, dtype, offset), dt)


def record(rows, q, v0, dv, dt, order, k, scan, offset=0):
    n = q.numel()
    traj = torch.empty((k + 1) * n + offset, dtype=q.dtype, device=DEV)[offset:]
    half = torch.empty(k * n, dtype=q.dtype, device=DEV) if dv is not None else None
    traj[:n] = q
    R.ram_step_record(rows, traj, half, v0, dv, dt, order, k, scan)
    return traj.view(k + 1, n), half


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("kind", ["uniform", "runs", "stretched", "huge", "dense"])
@pytest.mark.parametrize("n,offset", [(7, 0), (40, 0), (255, 0), (256, 1), (264, 0), (513, 0), (1024, 0),
                                      (1500, 0), (3001, 0)])
def test_alone_equals_planned(n, offset, kind, dtype):
    for with_dv in (True, False):
        rows, q, v0, dv, dt = inputs(n, kind, 5, with_dv, dtype, offset)
        order = 1 if kind in ("huge", "dense") else (3 if n % 2 else 5)
        for scan in SCANS[dtype]:
            t1, h1 = record(rows, q, v0, dv, dt, order, 1, scan, offset)
            t2, h2 = record(rows, q, v0, dv, dt, order, 2, scan, offset)
            torch.cuda.synchronize()
            assert torch.equal(t1[1], t2[1]), (with_dv, scan)
            assert h1 is None or torch.equal(h1, h2[:h1.numel()]), (with_dv, scan)
            if with_dv:
                continue
            out = torch.empty(q.numel() + offset, dtype=dtype, device=DEV)[offset:]
            R.ram_shift(rows, q, out, v0, dt, order, scan)
            torch.cuda.synchronize()
            assert torch.equal(out, t1[1]), scan


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("k", [1, 3, 5])
@pytest.mark.parametrize("n,offset", [(513, 0), (1024, 0), (1024, 1)])
def test_odd_steps_in_place(n, offset, k, dtype):
    rows, q, v0, dv, dt = inputs(n, "runs", 3, True, dtype, offset)
    traj, _ = record(rows, q, v0, dv, dt, 5, k, R.RAM_SUM_DIRECT, offset)
    R.ram_step(rows, q, v0, dv, dt, 5, k, R.RAM_SUM_DIRECT)
    torch.cuda.synchronize()
    assert torch.equal(q, traj[k])


@pytest.mark.parametrize("k", [1, 3, 5])
def test_odd_steps_elsewhere(k):
    # per-row meshes
    wl = W.small_ragged(7, 6, 900, seed=3, order=3)
    rows, q = R.Rows.from_workload(wl, DEV), dev(wl.q0, torch.float32)
    v0, dv = dev(wl.v0), dev(wl.dv, torch.float32)
    traj, _ = record(rows, q, v0, dv, wl.dt, 3, k, R.RAM_SUM_DIRECT)
    R.ram_step(rows, q, v0, dv, wl.dt, 3, k, R.RAM_SUM_DIRECT)
    torch.cuda.synchronize()
    assert torch.equal(q, traj[k])
    # limited steps, one call against k calls
    rows, q, v0, dv, dt = inputs(1023, "runs", 3, True, torch.float32, 0)
    one = q.clone()
    R.ram_step_limited(rows, q, v0, dv, dt, R.RAM_RECON_PPM, k)
    for _ in range(k):
        R.ram_step_limited(rows, one, v0, dv, dt, R.RAM_RECON_PPM, 1)
    torch.cuda.synchronize()
    assert torch.equal(q, one)
    # the reverse pass
    traj, half = record(rows, one, v0, dv, dt, 5, k, R.RAM_SUM_DIRECT)
    bar = dev(np.random.default_rng(2).standard_normal(3 * 1023), torch.float32)
    g = bar.clone()
    for i in reversed(range(k)):
        o = torch.empty_like(g)
        R.ram_step_adjoint(rows, traj[i], half[i * o.numel():(i + 1) * o.numel()], dv, g, o, v0, dt, 5)
        g = o
    R.ram_step_adjoint_steps(rows, traj, half, dv, bar, torch.empty_like(bar), v0, dt, 5, k)
    torch.cuda.synchronize()
    assert torch.equal(bar, g)


# FP32 batches of 65,536 tiles have a plan, one tile fewer none
@pytest.mark.parametrize("kind", ["runs", "stretched"])
def test_both_sides_of_the_plan(kind):
    n, few = 264, 32767                              # two tiles a row
    rng = np.random.default_rng(8)
    e = edges(kind, n)
    out = []
    q0 = torch.as_tensor(1.0 + 0.2 * rng.standard_normal((few + 1, n)), dtype=torch.float32, device=DEV)
    dv0 = torch.as_tensor(rng.uniform(-1, 1, (few + 1, n)), dtype=torch.float32, device=DEV)
    dt = 0.4 * float(np.diff(e).min())
    v0 = dev(rng.uniform(-0.7, 0.7, few + 1) / dt)
    for r in (few, few + 1):
        wl = W.Workload("plan", r, n, np.arange(r + 1) * n, e, True, np.zeros((0,)), None,
                        np.zeros(r), dt, 5, 1)
        q = q0[:r].reshape(-1).clone()
        R.ram_step(R.Rows.from_workload(wl, DEV), q, v0[:r].contiguous(),
                   dv0[:r].reshape(-1).contiguous(), dt, 5, 1, R.RAM_SUM_DIRECT)
        torch.cuda.synchronize()
        out.append(q.view(r, n))
    assert torch.equal(out[0], out[1][:few])


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("k", [1, 3, 5])
def test_odd_steps_with_a_schedule(k, dtype):
    rows, q, v0, dv, dt = inputs(1023, "runs", 3, True, dtype, 0)
    ctx = R.context(0)
    ctx.set_schedule(4)
    try:
        traj, _ = record(rows, q, v0, dv, dt, 5, k, R.RAM_SUM_DIRECT)
        R.ram_step(rows, q, v0, dv, dt, 5, k, R.RAM_SUM_DIRECT)
        torch.cuda.synchronize()
    finally:
        ctx.set_schedule(0)
    assert torch.equal(q, traj[k])
