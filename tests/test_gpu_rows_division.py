"""The per-row step's divisions, where an approximate quotient shows.

* Cells of 1 beside cells of 2^20 and 2^40 of the unit: at order 5 denominators of
  their stencils' outer weights pass FP32's largest number, and the weight is 0,
  as the quotient by infinity is.  (Every node is an integer, and no two nodes of
  a stencil round to one in FP32.)  With no shift every node lies on a mesh node,
  every weight is a product with 0, and a step returns the state to the rounding
  of (Q dx) / dx: two roundings, 2^-23 relative, doubled.  One step in each mode,
  four in one call (planned) by direct sums: prefix sums of such masses cancel.
* A reciprocal cell size that lies halfway between two FP32 numbers to FP64's last
  place, for 4096 sizes: what flows into an empty cell comes out as a quarter of
  the reciprocal rounded once, bit for bit.
* A shift of nothing: each cell is (Q dx) / dx in the type of the mode's sums,
  product and quotient rounded once each, bit for bit.
"""
import numpy as np
import pytest
import torch

from paper_2305_05362_amd import _lib as R

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


def dev(a, dtype=torch.float64):
    return torch.as_tensor(np.ascontiguousarray(a).reshape(-1), dtype=dtype, device=DEV)


@pytest.mark.parametrize("scan,steps", [(R.RAM_SCAN_F64, 1), (R.RAM_SCAN_F32_TWOSUM, 1), (R.RAM_SCAN_F32, 1),
                                        (R.RAM_SUM_DIRECT, 4)])
def test_weights_past_the_largest_number(scan, steps):
    w = np.exp2([0, 0, 0, 0, 20, 40, 40, 40, 40, 40, 40, 30, 20, 10])
    n, nr = len(w), 3
    e = np.concatenate([[0.0], np.cumsum(w)])
    rows = R.Rows(dev(np.tile(e, nr)), nr, n, None, False)
    q0 = np.random.default_rng(4).uniform(0.5, 2.0, n * nr).astype(np.float32)
    q = dev(q0, torch.float32)
    R.ram_step(rows, q, dev(np.zeros(nr)), None, 1.0, 5, steps, scan)
    got = q.cpu().numpy()
    assert np.isfinite(got).all(), np.argwhere(~np.isfinite(got)).ravel()
    assert np.max(np.abs(got / q0 - 1.0)) <= steps * 2.0 ** -22


def test_reciprocal_sizes_rounded_once():
    nr, n = 4096, 16
    i = np.random.default_rng(6).integers(0, 1 << 23, nr)
    dx = 1.0 / (1.0 + (2 * i + 1) * 2.0 ** -24)
    e = np.tile(np.arange(n + 1.0), (nr, 1))
    e[:, 1] = dx                                     # cell 0: from 0 to dx
    rows = R.Rows(dev(e), nr, n, None, False)
    q0, dv = np.zeros((nr, n)), np.zeros((nr, n))
    q0[:, -1] = 1.0
    dv[:, 0] = 1.0
    q = dev(q0, torch.float32)
    R.ram_step(rows, q, dev(np.zeros(nr)), dev(dv, torch.float32), 0.25, 5, 1, R.RAM_SCAN_F32_TWOSUM)
    got = q.cpu().numpy().reshape(nr, n)[:, 0]
    ref = np.float32(0.25) * (1.0 / dx).astype(np.float32)
    assert np.array_equal(got, ref), int((got != ref).sum())


@pytest.mark.parametrize("dtype,scan", [(torch.float64, R.RAM_SCAN_F64), (torch.float32, R.RAM_SCAN_F64),
                                        (torch.float32, R.RAM_SCAN_F32_TWOSUM), (torch.float32, R.RAM_SCAN_F32)])
@pytest.mark.parametrize("nr", [40, 600])
def test_mass_over_size(nr, dtype, scan):
    # (both tile sizes: batches of up to 393,216 cells and of more)
    n = 700
    rng = np.random.default_rng(8)
    e = np.concatenate([np.zeros((nr, 1)), np.cumsum(20.0 ** rng.random((nr, n)), axis=1)], axis=1)
    dx = np.diff(e, axis=1)
    q0 = rng.uniform(0.5, 2.0, (nr, n)).astype(np.float32)
    t = np.float64 if scan == R.RAM_SCAN_F64 else np.float32
    ref = (q0.astype(t) * dx.astype(t)) / dx.astype(t)
    rows = R.Rows(dev(e), nr, n, None, False)
    out = torch.empty(nr * n, dtype=dtype, device=DEV)
    R.ram_shift(rows, dev(q0, dtype), out, dev(np.zeros(nr)), 1.0, 5, scan)
    got = out.cpu().numpy().reshape(nr, n)
    ref = ref.astype(got.dtype)
    assert np.array_equal(got, ref), int((got != ref).sum())
