"""The tile adjoint (FP64; FP32 rows not a multiple of four cells) where a tile's
source window passes through LDS in pieces: rows refined tenfold (the periodic bump)
shifted anywhere in their period, and a row four fifths of whose cells lie in a
fourteenth of it, whose tiles take up to eighteen pieces; the last row shifted so
that nodes lie on nodes.

The streaming and the limited adjoint (FP32) on the same kind of row, whose windows
they take from global memory, with every node on a node but for the rounding of
v0 dt: where a plan and the kernel that reads it round a node's position differently,
it lies in two cells.

Against the oracle's residual and shift transposes at the bars of the tile adjoint's
tests; the dense row at order 1, whose error is a node's position, a few roundings
of the period in units of the smallest cell (64 eps L / dx_min of max |Q|).
"""
import numpy as np
import pytest
import torch

import oracle
from parity import CELL_F32_ADJ, assert_parity
from paper_2305_05362_amd import _lib as R
from paper_2305_05362_amd import workloads as W
from test_gpu_adjoint_tile import DEV, compare, dev, workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("with_dv", [True, False])
@pytest.mark.parametrize("n,order", [(1301, 5), (1602, 3), (2047, 5), (2050, 1), (3001, 5)])
def test_refined_rows(n, order, with_dv, dtype):
    e = W.bump_edges(n, -np.pi, np.pi, 0.2, 0.3, 9.0)
    compare(workload(n, e, order, with_dv, rows=8), dtype)


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("with_dv", [True, False])
def test_dozens_of_pieces(with_dv, dtype):
    w = np.concatenate([np.full(12000, 2.0 ** -6), np.ones(3001)])
    e = np.concatenate([[0.0], np.cumsum(w)])
    wl = workload(15001, e, 1, with_dv)
    wl.v0[2] = 7.0 / wl.dt
    bar = 64 * np.finfo(np.float64).eps * e[-1] / w.min()
    compare(wl, dtype, (bar, bar, 100 * bar) if dtype == torch.float64 else None)


def on_nodes():
    w = np.concatenate([np.full(1600, 2.0 ** -5), np.ones(1600)])
    e = np.concatenate([[0.0], np.cumsum(w)])
    wl = workload(3200, e, 1, False, rows=4)
    wl.dt = 0.1
    wl.v0 = np.array([3.0, -7.0, 1200.5, -801.25]) / wl.dt
    return wl


def test_streaming_adjoint_nodes_on_nodes():
    compare(on_nodes(), torch.float32)


@pytest.mark.parametrize("recon", [R.RAM_RECON_PLM, R.RAM_RECON_PPM])
def test_limited_adjoint_nodes_on_nodes(recon):
    wl = on_nodes()
    rbar = np.random.default_rng(4).standard_normal(wl.n_cells).astype(np.float32)
    qb = torch.empty(wl.n_cells, dtype=torch.float32, device=DEV)
    R.ram_shift_limited_adjoint(R.Rows.from_workload(wl, DEV), dev(wl.q0, torch.float32),
                                dev(rbar, torch.float32), qb, dev(wl.v0), wl.dt, recon)
    torch.cuda.synchronize()
    ref = oracle.shift_recon_adjoint(oracle.Rows.from_workload(wl), wl.q0.reshape(-1),
                                     rbar.astype(np.float64), wl.v0, wl.dt, recon)[0]
    assert_parity(qb.cpu().numpy().astype(np.float64), ref, 1e-5, CELL_F32_ADJ)
