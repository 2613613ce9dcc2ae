"""The FP32 streaming step on rows that are no multiple of four cells, or whose
arrays are not 16-byte aligned, and on either side of the tile count where both
kinds of tile go from one launch to two.

Where the word-aligned paths can go wrong: a row's first and last tile (the
neighbourhood crosses the row's end), a last tile of one, two, three or 255
cells, a window that crosses the row's end, rows shorter than a window, the
post-shift state's stores.  Against the oracle at the FP32 bars of one step
(1e-6 relative L1, CELL_F32 of max |Q| a cell).
"""
import numpy as np
import pytest
import torch

import oracle
from parity import CELL_F32, assert_parity
from paper_2305_05362_amd import _lib as R
from paper_2305_05362_amd import workloads as W

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


def dev(a, dtype=torch.float64, offset=0):
    a = torch.as_tensor(np.ascontiguousarray(a).reshape(-1), dtype=dtype)
    buf = torch.empty(a.numel() + offset, dtype=dtype, device=DEV)
    buf[offset:] = a.to(DEV)
    return buf[offset:]


def disk(n_r, n, mesh, dv=True):
    phi = None if mesh == "bump" else W.stretched_edges(n, 6.0, np.random.default_rng(n), -np.pi, np.pi)
    wl = W.polar(n_r, n, 2, 5, 1, name=f"{mesh}{n}", phi=phi)
    wl.q0 = wl.q0.astype(np.float32).astype(np.float64)
    wl.dv = wl.dv.astype(np.float32).astype(np.float64) if dv else None
    if not dv:
        wl.dt = 10.3 * 2 * np.pi / n / wl.v0.max()
    return wl


def check(wl, order, offset, rows=None):
    """One recorded step: the result and the post-shift state against the oracle."""
    n = wl.n_rows * wl.n_cols
    traj = torch.empty(2 * n + offset, dtype=torch.float32, device=DEV)[offset:]
    traj[:n] = dev(wl.q0, torch.float32)
    half = torch.empty(n + offset, dtype=torch.float32, device=DEV)[offset:]
    dv = None if wl.dv is None else dev(wl.dv, torch.float32, offset)
    R.ram_step_record(R.Rows.from_workload(wl, DEV), traj, half if dv is not None else None,
                      dev(wl.v0), dv, wl.dt, order, 1, R.RAM_SUM_DIRECT)
    torch.cuda.synchronize()
    pick = np.arange(wl.n_rows) if rows is None else np.asarray(rows)
    sub = W.Workload("sub", len(pick), wl.n_cols, W._uniform_row_ptr(len(pick), wl.n_cols), wl.edges,
                     True, wl.q0.reshape(wl.n_rows, -1)[pick], None, wl.v0[pick], wl.dt, order, 1)
    orows = oracle.Rows.from_workload(sub)
    mid = oracle.shift(orows, sub.q0, sub.v0, wl.dt, order)
    ref = mid
    if dv is not None:
        ref = oracle.residual(orows, mid, wl.dv.reshape(wl.n_rows, -1)[pick], wl.dt)
        got = half.cpu().numpy().reshape(wl.n_rows, -1)[pick]
        assert_parity(got, mid, 1e-6, CELL_F32, "half")
    got = traj[n:].cpu().numpy().reshape(wl.n_rows, -1)[pick]
    assert_parity(got, ref, 1e-6, CELL_F32, "step")


@pytest.mark.parametrize("n", [9, 131, 257, 259, 511, 1025, 2307])
@pytest.mark.parametrize("mesh", ["bump", "stretched"])
@pytest.mark.parametrize("order", [1, 5])
def test_odd_rows(n, mesh, order):
    check(disk(5, n, mesh), order, 0)
    check(disk(3, n, mesh, dv=False), order, 0)


@pytest.mark.parametrize("offset", [1, 2, 3])
@pytest.mark.parametrize("mesh", ["bump", "stretched"])
def test_unaligned_arrays(offset, mesh):
    check(disk(4, 1024, mesh), 5, offset)
    check(disk(4, 1026, mesh, dv=False), 3, offset)


# 32767 tiles (one launch) and 32774 (two)
@pytest.mark.parametrize("n_r", [4681, 4682])
@pytest.mark.parametrize("mesh", ["bump", "stretched"])
def test_both_sides_of_one_launch(n_r, mesh):
    check(disk(n_r, 7 * 256 - 4, mesh), 5, 0, rows=[0, 1, n_r // 2, n_r - 2, n_r - 1])
