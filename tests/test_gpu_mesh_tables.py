"""The shared mesh's tables at the sizes where their kernel splits its work:
workgroups of 256 and 512 threads (rows up to and beyond 4096 cells), the run
counts kept in registers or re-read (4, 12, 16, 32 cells a lane), buckets whose
cells lie beyond the wave's 128-node window (a mesh graded a thousandfold, most
of whose cells fall in few buckets).

* FP64 shifts by many cells against the oracle, on noisy states, where a wrong
  bucket or stencil moves a cell's value by the noise (0.05).  Bar per cell: a
  node's position carries a few roundings of the period (eps L), which in
  units of the smallest cell is eps L / dx_min, times the weights' and the
  state's size: 64 eps L / dx_min of max |Q|, 3e-8 on the finest mesh here.
* The path of every tile at zero shift on a uniform mesh with one cell off:
  uniform exactly where neither the tile's cells (one beyond each end) nor its
  source window hold the odd cell.
"""
import numpy as np
import pytest
import torch

import oracle
from parity import max_cell
from paper_2305_05362_amd import _lib as R
from paper_2305_05362_amd import workloads as W

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


def dev(a, dtype=torch.float64):
    return torch.as_tensor(np.ascontiguousarray(a).reshape(-1), dtype=dtype, device=DEV)


def graded(n, ratio):
    w = ratio ** (np.arange(n) / n)
    e = np.concatenate([[0.0], np.cumsum(w)])
    e /= e[-1]
    e[-1] = 1.0
    return e


# (graded a thousandfold only over rows long enough that neighbouring cells
# stay within a few percent of each other: the FP64 bars assume it)
@pytest.mark.parametrize("ratio,n", [(8.0, n) for n in (6, 64, 255, 257, 1025, 4096, 4097, 16384,
                                                        16387)] +
                         [(1000.0, n) for n in (255, 257, 1025, 4096, 4097, 16384, 16387)])
def test_shift_on_graded_mesh(ratio, n):
    e = graded(n, ratio)
    rng = np.random.default_rng(n)
    q = 1.0 + W.sine_cell_averages(e, 0.0, 0.3, 2, 0.4) + 0.05 * rng.standard_normal(n)
    q = np.stack([q, q[::-1]])
    v0 = np.array([0.3173, -4.0 / n])
    wl = W.Workload("graded", 2, n, W._uniform_row_ptr(2, n), e, True, q, None, v0, 1.0, 5, 1)
    rows = R.Rows.from_workload(wl, DEV)
    out = torch.empty(2 * n, dtype=torch.float64, device=DEV)
    R.ram_shift(rows, dev(q), out, dev(v0), 1.0, 5)
    torch.cuda.synchronize()
    ref = oracle.shift(oracle.Rows.from_workload(wl), q, v0, 1.0, 5)
    err = max_cell(out.cpu().numpy(), ref)
    assert err <= 64 * np.finfo(np.float64).eps / np.diff(e).min(), (n, err)


@pytest.mark.parametrize("n", [1024, 1025, 2100, 4096, 4097, 6145, 16384, 16640])
def test_tile_paths_around_one_cell(n):
    order, lo = 5, 2
    for odd in (0, 700, n - 1):
        w = np.full(n, 1.0 / n)
        w[odd] *= 1.01
        e = np.concatenate([[0.0], np.cumsum(w)])
        rows = R.Rows(dev(e), 1, n, None, True)
        got = R.context(0).ram_step_tile_paths(rows, dev(np.zeros(1)), 1.0, order, False)
        want = []
        for i0 in range(0, n, 256):
            nd = min(256, n - i0)
            hit = any((odd - a) % n < b - a for a, b in ((i0 - 1, i0 + nd + 1),
                                                         (i0 - lo, i0 - lo + nd + order)))
            want.append(R.RAM_TILE_WINDOW if hit else R.RAM_TILE_UNIFORM)
        assert got.cpu().tolist() == want, (n, odd)


# rows whose run counts are shared out over workgroups (beyond 16384 cells; from two
# million on as many as there are), odd cells around the edges of their segments and waves
@pytest.mark.parametrize("n", [16385, 20480, 33000, 100001, (1 << 20) + 3, (1 << 21) + 4097])
def test_tile_paths_on_long_rows(n):
    order, lo = 5, 2
    rng = np.random.default_rng(n)
    odd = np.unique(np.concatenate([[0, n - 1, 511, 512, 4095, 4096, 4097, n // 2],
                                    rng.integers(0, n, 40)]))
    for size in (1.01, 0.99):                        # beside the smallest, beside the largest
        w = np.ones(n)
        w[odd] = size
        e = np.concatenate([[0.0], np.cumsum(w)])
        rows = R.Rows(dev(e), 1, n, None, True)
        got = R.context(0).ram_step_tile_paths(rows, dev(np.zeros(1)), 1.0, order, False).cpu().numpy()
        i0 = np.arange(0, n, 256)
        nd = np.minimum(256, n - i0)
        # (from the sizes as the nodes have them: past a million cells the nodes' own
        # rounding passes the tolerance of 1e-10 here and there)
        d = np.diff(e)
        uniform = np.zeros(len(i0), dtype=bool)
        for h in (d.max(), d.min()):
            flag = (np.abs(d - h) > 1e-10 * h).astype(np.int64)
            count = np.concatenate([[0], np.cumsum(np.tile(flag, 3))])
            uniform |= ((count[n + i0 + nd + 1] - count[n + i0 - 1]) +
                        (count[n + i0 - lo + nd + order] - count[n + i0 - lo])) == 0
        want = np.where(uniform, R.RAM_TILE_UNIFORM, R.RAM_TILE_WINDOW)
        assert np.array_equal(got, want), (n, size, np.argwhere(got != want).ravel()[:10])


# the same where one workgroup counts, its lanes' cells flagged as bits (12 and 32 a lane)
@pytest.mark.parametrize("n", [4100, 6144, 6145, 12001, 16384])
def test_tile_paths_of_one_workgroups_counts(n):
    test_tile_paths_on_long_rows(n)
