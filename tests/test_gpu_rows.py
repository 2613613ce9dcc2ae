"""The per-row step where its wave tiles can go wrong: rows of 6 cells up (a
window that crosses the row's end twice), one cell less, as many and one more
than a tile holds (251 with the residual, 255 without, and their multiples),
windows beyond the LDS (a row half of whose cells lie in a hundredth of it), and
a batch of more rows than one pass of the tile table's fill covers.

FP64 and FP32 against the oracle at the bars the ragged tests use (FP64 1e-12
relative L1 and CELL_F64; FP32 1e-6 and 2e-4 of max |Q| a cell); the dense row
at order 1, whose error is a node's position, a few roundings of the period in
units of the smallest cell (64 eps L / dx_min of max |Q|).
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
LENS = [6, 7, 8, 9, 10, 13, 40, 250, 251, 252, 254, 255, 256, 257, 502, 503, 510, 511, 1020, 1021, 1500]


def dev(a, dtype=torch.float64):
    return torch.as_tensor(np.ascontiguousarray(a).reshape(-1), dtype=dtype, device=DEV)


def batch(lens, order, with_dv, seed, ratio=20.0, edges=None):
    rng = np.random.default_rng(seed)
    lens = np.asarray(lens, dtype=np.int64)
    ptr = np.concatenate([[0], np.cumsum(lens)])
    es = edges or [W.stretched_edges(int(n), ratio, rng) for n in lens]
    q = np.concatenate([1.0 + W.sine_cell_averages(e, 0.0, 0.3, 2, 0.3) +
                        0.05 * rng.standard_normal(len(e) - 1) for e in es])
    q = q.astype(np.float32).astype(np.float64)
    dv, dt = None, 1.0
    if with_dv:
        dv = (0.3 * rng.standard_normal(len(q))).astype(np.float32).astype(np.float64)
        dt = min(W.residual_cfl_dt(e, dv[ptr[r]:ptr[r + 1]][None, :], 0.5) for r, e in enumerate(es))
    v0 = rng.uniform(-30.0, 30.0, len(lens)) / lens / dt
    return W.Workload("rows", len(lens), 0, ptr, np.concatenate(es), False, q, dv, v0, dt, order, 1)


def run(wl, dtype, scan):
    rows = R.Rows.from_workload(wl, DEV)
    q = dev(wl.q0, dtype)
    R.ram_step(rows, q, dev(wl.v0), None if wl.dv is None else dev(wl.dv, dtype), wl.dt, wl.order, 1, scan)
    torch.cuda.synchronize()
    ref = oracle.step(oracle.Rows.from_workload(wl), wl.q0, wl.v0, wl.dv, wl.dt, wl.order, 1)
    return q.cpu().numpy().astype(np.float64), ref


@pytest.mark.parametrize("order", [1, 3, 5])
@pytest.mark.parametrize("with_dv", [True, False])
@pytest.mark.parametrize("dtype,scan", [(torch.float64, R.RAM_SCAN_F64), (torch.float32, R.RAM_SCAN_F64),
                                        (torch.float32, R.RAM_SCAN_F32_TWOSUM)])
def test_row_lengths(order, with_dv, dtype, scan):
    got, ref = run(batch(LENS, order, with_dv, 5), dtype, scan)
    if dtype == torch.float64:
        assert_parity(got, ref, 1e-12, CELL_F64)
    else:
        assert_parity(got, ref, 1e-6, 2e-4)


# the same in a batch of more than 393,216 cells (four node slots a lane, where a
# small batch has two) and around the two slots' tiles (123 and 127 cells)
@pytest.mark.parametrize("with_dv", [True, False])
@pytest.mark.parametrize("dtype,scan", [(torch.float64, R.RAM_SCAN_F64), (torch.float32, R.RAM_SCAN_F64),
                                        (torch.float32, R.RAM_SCAN_F32_TWOSUM)])
@pytest.mark.parametrize("more", [0, 290])
def test_both_tile_sizes(more, with_dv, dtype, scan):
    lens = LENS + [122, 123, 124, 126, 127, 128, 246, 247, 381, 382] + [1400] * more
    got, ref = run(batch(lens, 3, with_dv, 11), dtype, scan)
    if dtype == torch.float64:
        assert_parity(got, ref, 1e-12, CELL_F64)
    else:
        assert_parity(got, ref, 1e-6, 2e-4)


@pytest.mark.parametrize("with_dv", [True, False])
@pytest.mark.parametrize("steps", [1, 4])
def test_windows_beyond_the_lds(with_dv, steps):
    # a tile of the coarse half takes its cells from the dense one
    w = np.concatenate([np.full(750, 1e-2), np.ones(750)])
    e = np.concatenate([[0.0], np.cumsum(w)]) / w.sum()
    e[-1] = 1.0
    wl = batch([1500] * 3, 1, with_dv, 9, edges=[e] * 3)
    wl.v0 = np.array([0.004, 0.3, -0.45]) / wl.dt
    wl.steps = steps
    rows = R.Rows.from_workload(wl, DEV)
    for dtype in (torch.float64, torch.float32):
        q = dev(wl.q0, dtype)
        R.ram_step(rows, q, dev(wl.v0), None if wl.dv is None else dev(wl.dv, dtype), wl.dt, 1, steps,
                   R.RAM_SCAN_F64)
        torch.cuda.synchronize()
        ref = oracle.step(oracle.Rows.from_workload(wl), wl.q0, wl.v0, wl.dv, wl.dt, 1, steps)
        err = max_cell(q.cpu().numpy(), ref)
        bar = 64 * np.finfo(np.float64).eps / np.diff(e).min() * steps
        assert err <= (bar if dtype == torch.float64 else 2e-4), (dtype, err, bar)


def test_more_rows_than_one_fill():
    lens = np.random.default_rng(3).integers(6, 30, 8300)
    lens[::1000] = 600
    got, ref = run(batch(lens, 3, False, 7, ratio=4.0), torch.float64, R.RAM_SCAN_F64)
    assert_parity(got, ref, 1e-12, CELL_F64)
