"""The per-row step where a tile's source window passes through LDS in pieces: rows
refined tenfold (the periodic bump), shifted anywhere in their period, in batches
of both tile sizes; rows of a few cells whose windows cross the row's end more than
twice; a row half of whose cells lie in a thousandth of it (dozens of pieces a
tile), shifted so that nodes lie on its nodes too.

Against the oracle at the bars of the ragged tests (FP64 1e-12 relative L1 and
CELL_F64; FP32 1e-6 and 2e-4 of max |Q| a cell); the dense row at order 1, whose
error is a node's position, a few roundings of the period in units of the smallest
cell (64 eps L / dx_min of max |Q|).  The recorded half step and the plain step
agree bit for bit.
"""
import numpy as np
import pytest
import torch

import oracle
from parity import CELL_F64, assert_parity, max_cell
from paper_2305_05362_amd import _lib as R
from paper_2305_05362_amd import workloads as W

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")
MODES = [(torch.float64, R.RAM_SCAN_F64), (torch.float32, R.RAM_SCAN_F64), (torch.float32, R.RAM_SCAN_F32_TWOSUM)]


def dev(a, dtype=torch.float64):
    return torch.as_tensor(np.ascontiguousarray(a).reshape(-1), dtype=dtype, device=DEV)


def bump(n):
    return W.bump_edges(n, -np.pi, np.pi, 0.2, 0.3, 9.0)


def workload(edges, nr, order, with_dv, seed):
    rng = np.random.default_rng(seed)
    n = len(edges) - 1
    e = np.tile(edges, (nr, 1))
    q = 1.0 + 0.3 * np.sin(2 * np.pi * np.arange(n) / n)[None, :] + 0.05 * rng.standard_normal((nr, n))
    q = q.astype(np.float32).astype(np.float64)
    dv, dt = None, 1.0
    if with_dv:
        dv = (0.3 * rng.standard_normal((nr, n))).astype(np.float32).astype(np.float64)
        dt = W.residual_cfl_dt(edges, dv, 0.5)
    v0 = rng.uniform(-1.5, 1.5, nr) * (edges[-1] - edges[0]) / dt
    return W.Workload("wide", nr, n, np.arange(nr + 1) * n, e, False, q, dv, v0, dt, order, 1)


def step(wl, dtype, scan):
    rows = R.Rows.from_workload(wl, DEV)
    q = dev(wl.q0, dtype)
    dv = None if wl.dv is None else dev(wl.dv, dtype)
    traj = torch.empty((2, q.numel()), dtype=dtype, device=DEV)
    half = torch.empty((1, q.numel()), dtype=dtype, device=DEV) if dv is not None else None
    traj[0] = q
    R.ram_step(rows, q, dev(wl.v0), dv, wl.dt, wl.order, 1, scan)
    R.ram_step_record(rows, traj, half, dev(wl.v0), dv, wl.dt, wl.order, 1, scan)
    torch.cuda.synchronize()
    assert torch.equal(traj[1], q)
    return q.cpu().numpy().astype(np.float64)


def check(wl, dtype, scan):
    ref = oracle.step(oracle.Rows.from_workload(wl), wl.q0.reshape(-1), wl.v0,
                      None if wl.dv is None else wl.dv.reshape(-1), wl.dt, wl.order, 1)
    got = step(wl, dtype, scan)
    if dtype == torch.float64:
        assert_parity(got, ref, 1e-12, CELL_F64)
    else:
        assert_parity(got, ref, 1e-6, 2e-4)


@pytest.mark.parametrize("with_dv", [True, False])
@pytest.mark.parametrize("dtype,scan", MODES)
@pytest.mark.parametrize("n,nr,order", [(700, 20, 5), (1000, 20, 3), (2000, 20, 5), (2001, 20, 1), (700, 600, 5),
                                        (1499, 300, 3)])
def test_refined_rows(n, nr, order, dtype, scan, with_dv):
    check(workload(bump(n), nr, order, with_dv, n + nr), dtype, scan)


# two cells thirty times the other five: the two cells a side that a
# tile's halo adds take it round the row again
@pytest.mark.parametrize("with_dv", [True, False])
@pytest.mark.parametrize("dtype,scan", MODES)
def test_short_rows_round_their_end(dtype, scan, with_dv):
    w = np.array([30.0, 30.0] + [1.0] * 5)
    e = np.concatenate([[0.0], np.cumsum(w)]) / w.sum()
    e[-1] = 1.0
    check(workload(e, 40, 1, with_dv, 7), dtype, scan)


@pytest.mark.parametrize("with_dv", [True, False])
def test_dozens_of_pieces(with_dv):
    w = np.concatenate([np.full(10000, 2.0 ** -10), np.ones(10000)])
    e = np.concatenate([[0.0], np.cumsum(w)])
    wl = workload(e, 4, 1, with_dv, 3)
    # node on node (a sum of cells of either kind), and anywhere
    wl.v0 = np.array([5.0, 2.0 ** -9, 3210.123, -777.7]) / wl.dt
    ref = oracle.step(oracle.Rows.from_workload(wl), wl.q0.reshape(-1), wl.v0,
                      None if wl.dv is None else wl.dv.reshape(-1), wl.dt, 1, 1)
    bar = 64 * np.finfo(np.float64).eps * e[-1] / np.diff(e).min()
    for dtype, scan in MODES:
        err = max_cell(step(wl, dtype, scan), ref)
        assert err <= (bar if dtype == torch.float64 else 2e-4), (dtype, err, bar)
