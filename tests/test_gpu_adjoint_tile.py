"""The tile adjoint (FP64; FP32 rows not a multiple of four cells) where it can
go wrong: the shortest row it takes (a tile and a halo), one cell more and less
than whole tiles, a last tile of one cell, windows beyond the LDS, and nodes
that share a source cell (one LDS turn each), up to a cell of six tenths of the
period, which a node lies in further than half a period from its edge.

Against the oracle's residual and shift transposes, at the bars of the step
adjoint's tests: FP64 1e-12 relative L1 and CELL_F64, v0bar 1e-10 of its
largest; FP32 1e-5, CELL_F32_ADJ and 1e-3.  The meshes with a huge cell run at
order 1, where the error is a node's position, a few roundings of the period in
units of the smallest cell: 64 eps L / dx_min of max |Q| (FP32: the FP32 bars).
The limited adjoint on that mesh at the FP32 bars.  The steps call equals
one-step calls bit for bit.
"""
import numpy as np
import pytest
import torch

import oracle
from parity import CELL_F32_ADJ, CELL_F64, assert_parity, max_cell
from paper_2305_05362_amd import _lib as R
from paper_2305_05362_amd import workloads as W

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


def dev(a, dtype=torch.float64):
    return torch.as_tensor(np.ascontiguousarray(a).reshape(-1), dtype=dtype, device=DEV)


def workload(n, edges, order, with_dv, rows=3, seed=2):
    rng = np.random.default_rng(seed + n)
    q = 1.0 + 0.3 * np.sin(2 * np.pi * np.arange(n) / n)[None, :] + 0.05 * rng.standard_normal((rows, n))
    dv, dt = None, 1.0
    if with_dv:
        dv = rng.uniform(-1, 1, (rows, n)).astype(np.float32).astype(np.float64)
        dt = W.residual_cfl_dt(edges, dv, 0.5)
    v0 = rng.uniform(-0.7, 0.7, rows) * (edges[-1] - edges[0]) / dt
    return W.Workload("tile", rows, n, np.arange(rows + 1) * n, edges, True,
                      q.astype(np.float32).astype(np.float64), dv, v0, dt, order, 1)


def reference(wl, qh, rbar):
    orows = oracle.Rows.from_workload(wl)
    dvb = None
    if wl.dv is not None:
        rbar, dvb = oracle.residual_adjoint(orows, qh, wl.dv.reshape(-1), rbar, wl.dt)
    qb, v0b = oracle.shift_adjoint(orows, wl.q0.reshape(-1), rbar, wl.v0, wl.dt, wl.order)
    return qb, dvb, v0b


def compare(wl, dtype, bars=None):
    n = wl.n_cells
    rng = np.random.default_rng(n)
    qh = oracle.shift(oracle.Rows.from_workload(wl), wl.q0.reshape(-1), wl.v0, wl.dt, wl.order)
    qh = qh.astype(np.float32).astype(np.float64)
    rbar = rng.standard_normal(n).astype(np.float32).astype(np.float64)
    rows = R.Rows.from_workload(wl, DEV)
    has = wl.dv is not None
    qb = torch.full((n,), float("nan"), dtype=dtype, device=DEV)
    dvb = torch.zeros(n, dtype=dtype, device=DEV) if has else None
    v0b = torch.zeros(wl.n_rows, dtype=torch.float64, device=DEV)
    args = (dev(wl.q0, dtype), dev(qh, dtype) if has else None, dev(wl.dv, dtype) if has else None)
    R.ram_step_adjoint(rows, *args, dev(rbar, dtype), qb, dev(wl.v0), wl.dt, wl.order, dvb, v0b)
    torch.cuda.synchronize()
    ref = reference(wl, qh, rbar)
    f64 = dtype == torch.float64
    l1, cell, v = bars or ((1e-12, CELL_F64, 1e-10) if f64 else (1e-5, CELL_F32_ADJ, 1e-3))
    got = qb.cpu().numpy().astype(np.float64)
    assert_parity(got, ref[0], l1, cell, what="qbar")
    if has:
        assert_parity(dvb.cpu().numpy().astype(np.float64), ref[1], l1, cell, what="dvbar")
    assert np.max(np.abs(v0b.cpu().numpy() - ref[2])) <= v * np.max(np.abs(ref[2]))
    # without v0bar (another kernel of the family): the same gradient
    qb2 = torch.empty_like(qb)
    R.ram_step_adjoint(rows, None, *args[1:], dev(rbar, dtype), qb2, dev(wl.v0), wl.dt, wl.order)
    torch.cuda.synchronize()
    assert_parity(qb2.cpu().numpy().astype(np.float64), ref[0], l1, cell, what="qbar alone")


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("with_dv", [True, False])
@pytest.mark.parametrize("order", [1, 3, 5])
@pytest.mark.parametrize("n", [264, 265, 511, 512, 513, 770, 1023])
def test_row_lengths(n, order, with_dv, dtype):
    if dtype == torch.float32 and n % 4 == 0:
        n += 2
    e = W.stretched_edges(n, 8.0, np.random.default_rng(n))
    compare(workload(n, e, order, with_dv), dtype)
    compare(workload(n, W.uniform_edges(n, 0.0, 1.0), order, with_dv), dtype)


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("with_dv", [True, False])
@pytest.mark.parametrize("kind", ["huge", "dense"])
def test_shared_cells_and_wide_windows(kind, with_dv, dtype):
    w = np.ones(1501)
    if kind == "huge":
        w[700] = 2250.0                              # six tenths of the period
    else:
        w[:1200] = 0.02                              # windows of up to 1200 cells
    e = np.concatenate([[0.0], np.cumsum(w)]) / w.sum()
    e[-1] = 1.0
    wl = workload(1501, e, 1, with_dv)
    bar = 64 * np.finfo(np.float64).eps / np.diff(e).min()
    compare(wl, dtype, (bar, bar, 100 * bar) if dtype == torch.float64 else None)
    if dtype == torch.float64:                       # the forward step on the same mesh
        q = dev(wl.q0)
        R.ram_step(R.Rows.from_workload(wl, DEV), q, dev(wl.v0),
                   dev(wl.dv) if with_dv else None, wl.dt, 1, 1, R.RAM_SUM_DIRECT)
        torch.cuda.synchronize()
        ref = oracle.step(oracle.Rows.from_workload(wl), wl.q0.reshape(-1), wl.v0,
                          wl.dv.reshape(-1) if with_dv else None, wl.dt, 1, 1)
        assert max_cell(q.cpu().numpy(), ref) <= bar


@pytest.mark.parametrize("dtype,n", [(torch.float64, 1024), (torch.float32, 1021)])
def test_steps_equal_single_steps(dtype, n):
    wl = workload(n, W.stretched_edges(n, 8.0, np.random.default_rng(n)), 5, True)
    rows = R.Rows.from_workload(wl, DEV)
    k = 3
    traj = torch.empty((k + 1, wl.n_cells), dtype=dtype, device=DEV)
    half = torch.empty((k, wl.n_cells), dtype=dtype, device=DEV)
    traj[0] = dev(wl.q0, dtype)
    v0, dv = dev(wl.v0), dev(wl.dv, dtype)
    R.ram_step_record(rows, traj, half, v0, dv, wl.dt, 5, k, R.RAM_SCAN_F64)
    bar = dev(np.random.default_rng(1).standard_normal(wl.n_cells), dtype)
    one, dv1, s1 = bar.clone(), torch.zeros_like(bar), torch.zeros(3, dtype=torch.float64, device=DEV)
    for i in reversed(range(k)):
        out = torch.empty_like(one)
        R.ram_step_adjoint(rows, traj[i], half[i], dv, one, out, v0, wl.dt, 5, dv1, s1)
        one = out
    many, dv2, s2 = bar.clone(), torch.zeros_like(bar), torch.zeros_like(s1)
    R.ram_step_adjoint_steps(rows, traj, half, dv, many, torch.empty_like(many), v0, wl.dt, 5, k,
                             dv2, s2)
    torch.cuda.synchronize()
    assert torch.equal(one, many) and torch.equal(dv1, dv2) and torch.equal(s1, s2)


@pytest.mark.parametrize("recon", [R.RAM_RECON_PLM, R.RAM_RECON_PPM])
def test_limited_adjoint_huge_cell(recon):
    w = np.ones(1500)
    w[700] = 2250.0
    e = np.concatenate([[0.0], np.cumsum(w)]) / w.sum()
    e[-1] = 1.0
    wl = workload(1500, e, 3, False)
    rbar = np.random.default_rng(4).standard_normal(wl.n_cells).astype(np.float32)
    qb = torch.empty(wl.n_cells, dtype=torch.float32, device=DEV)
    R.ram_shift_limited_adjoint(R.Rows.from_workload(wl, DEV), dev(wl.q0, torch.float32),
                                dev(rbar, torch.float32), qb, dev(wl.v0), wl.dt, recon)
    torch.cuda.synchronize()
    ref = oracle.shift_recon_adjoint(oracle.Rows.from_workload(wl), wl.q0.reshape(-1),
                                     rbar.astype(np.float64), wl.v0, wl.dt, recon)[0]
    assert_parity(qb.cpu().numpy().astype(np.float64), ref, 1e-5, CELL_F32_ADJ)
