"""The tile adjoint (FP64; FP32 rows not a multiple of four cells) where a tile's
source window passes through LDS in pieces: rows refined tenfold (the periodic bump)
shifted anywhere in their period, and a row four fifths of whose cells lie in a
fourteenth of it, whose tiles take up to eighteen pieces; the last row shifted so
that nodes lie on nodes.

Against the oracle's residual and shift transposes at the bars of the tile adjoint's
tests; the dense row at order 1, whose error is a node's position, a few roundings
of the period in units of the smallest cell (64 eps L / dx_min of max |Q|).
"""
import numpy as np
import pytest
import torch

from paper_2305_05362_amd import workloads as W
from test_gpu_adjoint_tile import compare, workload

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
