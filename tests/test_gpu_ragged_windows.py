"""The streaming step on per-row meshes (FP32, no residual, four steps and more)
where the way a window's masses are accumulated changes: windows of one slot of the
wave (64 cells), of up to five slots (320), and more.  Rows of a tile and less, whose
windows hold the row and its stencil, around both lines; two tiles and more.

Against the oracle at the bars of the ragged streaming tests (1e-6 relative L1, 2e-4
of max |Q| a cell, for four steps).
"""
import numpy as np
import pytest
import torch

import oracle
from parity import assert_parity
from paper_2305_05362_amd import _lib as R
from paper_2305_05362_amd import workloads as W

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")
LENS = [6, 7, 12, 20, 57, 58, 59, 60, 61, 62, 63, 64, 65, 66, 120, 254, 255, 256, 311, 315, 316, 320, 321,
        510, 700]


@pytest.mark.parametrize("order", [1, 3, 5])
@pytest.mark.parametrize("scan", [R.RAM_SCAN_F64, R.RAM_SCAN_F32_TWOSUM, R.RAM_SUM_DIRECT])
def test_windows(scan, order):
    rng = np.random.default_rng(12)
    lens = np.array(LENS, dtype=np.int64)
    ptr = np.concatenate([[0], np.cumsum(lens)])
    es = [W.stretched_edges(int(n), 4.0, rng) for n in lens]
    q = np.concatenate([1.0 + W.sine_cell_averages(e, 0.0, 0.3, 1, 0.3) for e in es])
    q = q.astype(np.float32).astype(np.float64)
    v0 = rng.uniform(-0.9, 0.9, len(lens))
    wl = W.Workload("windows", len(lens), 0, ptr, np.concatenate(es), False, q, None, v0, 1.0, order, 4)
    s = torch.as_tensor(q, dtype=torch.float32, device=DEV)
    R.ram_step(R.Rows.from_workload(wl, DEV), s, torch.as_tensor(v0, device=DEV), None, 1.0, order, 4, scan)
    torch.cuda.synchronize()
    ref = oracle.step(oracle.Rows.from_workload(wl), q, v0, None, 1.0, order, 4)
    assert_parity(s.cpu().numpy().astype(np.float64), ref, 1e-6, 2e-4)


# rows of a few cells take the window like any other, in the arithmetic that their mode
# names: with no shift every weight is 0, and a step is (Q dx) / dx in FP32, bit for bit
@pytest.mark.parametrize("steps,scan", [(1, R.RAM_SCAN_F32_TWOSUM), (1, R.RAM_SCAN_F32), (4, R.RAM_SUM_DIRECT)])
@pytest.mark.parametrize("n,order", [(4, 3), (6, 1), (6, 5), (7, 5), (8, 3), (9, 5), (10, 5)])
def test_rows_of_a_few_cells(n, order, scan, steps):
    nr = 500
    rng = np.random.default_rng(n)
    e = np.concatenate([np.zeros((nr, 1)), np.cumsum(rng.uniform(1, 3, (nr, n)), axis=1)], axis=1)
    dx = np.diff(e, axis=1).astype(np.float32)
    q0 = rng.uniform(0.5, 2.0, (nr, n)).astype(np.float32)
    q = torch.as_tensor(q0.reshape(-1), device=DEV)
    rows = R.Rows(torch.as_tensor(e.reshape(-1), device=DEV), nr, n, None, False)
    R.ram_step(rows, q, torch.zeros(nr, dtype=torch.float64, device=DEV), None, 1.0, order, steps, scan)
    ref = q0
    for _ in range(steps):
        ref = (ref * dx) / dx
    got = q.cpu().numpy().reshape(nr, n)
    assert np.array_equal(got, ref), int((got != ref).sum())


# the tile table: one workgroup up to 8192 rows of eight tiles each, else all share the fill
@pytest.mark.parametrize("nr,tall", [(1, 6), (3000, 20), (3000, 1016), (3000, 1017), (8192, 30), (8193, 30),
                                     (2000, 9000)])
def test_tile_table(nr, tall):
    rng = np.random.default_rng(nr + tall)
    lens = rng.integers(6, 20, nr)
    lens[nr // 2] = tall
    ptr = np.concatenate([[0], np.cumsum(lens)])
    es = [W.stretched_edges(int(n), 2.0, rng) for n in lens]
    q = rng.uniform(0.5, 2.0, int(ptr[-1]))
    v0 = rng.uniform(-0.9, 0.9, nr)
    wl = W.Workload("table", nr, 0, ptr, np.concatenate(es), False, q, None, v0, 1.0, 1, 1)
    out = torch.empty(len(q), dtype=torch.float64, device=DEV)
    R.ram_shift(R.Rows.from_workload(wl, DEV), torch.as_tensor(q, device=DEV), out,
                torch.as_tensor(v0, device=DEV), 1.0, 1)
    ref = oracle.shift(oracle.Rows.from_workload(wl), q, v0, 1.0, 1)
    assert_parity(out.cpu().numpy(), ref, 1e-12, 1e-11)
