"""ram_shift_noalloc on per-row meshes takes ram_shift's tiles: equal to it bit for
bit in the prefix modes too, whose roundings go by the tile, in batches of both tile
sizes (up to 393,216 cells and more), up to the rows that just fit the static buffer
(16 MiB: 32 bytes a row and one for every 42 cells)."""
import numpy as np
import pytest
import torch

from paper_2305_05362_amd import _lib as R
from paper_2305_05362_amd import workloads as W

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


def dev(a, dtype=torch.float64):
    return torch.as_tensor(np.ascontiguousarray(a).reshape(-1), dtype=dtype, device=DEV)


@pytest.mark.parametrize("dtype,scan", [(torch.float64, R.RAM_SCAN_F64), (torch.float32, R.RAM_SUM_DIRECT),
                                        (torch.float32, R.RAM_SCAN_F32_TWOSUM), (torch.float32, R.RAM_SCAN_F32)])
@pytest.mark.parametrize("rows,lo,hi", [(40, 8, 2600), (3000, 6, 40), (500, 600, 1300), (1, 9, 9)])
def test_equals_shift(rows, lo, hi, dtype, scan):
    wl = W.small_ragged(rows, lo, hi, seed=rows, order=5)
    r = R.Rows.from_workload(wl, DEV)
    q, v0 = dev(wl.q0, dtype), dev(wl.v0)
    a, b = torch.full_like(q, float("nan")), torch.full_like(q, float("nan"))
    ctx = R.context(0)
    ctx.ram_shift_noalloc(r, q, a, v0, wl.dt, 5, scan)
    ctx.ram_shift(r, q, b, v0, wl.dt, 5, scan)
    torch.cuda.synchronize()
    assert torch.isfinite(b).all() and torch.equal(a, b)


def test_rows_that_just_fit():
    n, nr = 7, 521000
    rng = np.random.default_rng(1)
    e = np.tile(np.concatenate([[0.0], np.cumsum(rng.uniform(1, 3, n))]), (nr + 1, 1))
    q0 = rng.uniform(0.5, 2.0, (nr + 1) * n)
    v = rng.uniform(-20, 20, nr + 1)
    ctx = R.context(0)
    for k, fits in ((nr, True), (nr + 1000, False)):
        ptr = torch.arange(k + 1, dtype=torch.int64, device=DEV) * n
        rows = R.Rows(dev(np.resize(e, (k, n + 1))), k, 0, ptr, False, k * n)
        q, v0 = dev(np.resize(q0, k * n), torch.float32), dev(np.resize(v, k))
        a, b = torch.full_like(q, float("nan")), torch.full_like(q, float("nan"))
        if not fits:
            with pytest.raises(R.RamError) as ei:
                ctx.ram_shift_noalloc(rows, q, a, v0, 1.0, 5, R.RAM_SCAN_F32_TWOSUM)
            assert ei.value.status == R.RAM_E_NOMEM
            continue
        ctx.ram_shift_noalloc(rows, q, a, v0, 1.0, 5, R.RAM_SCAN_F32_TWOSUM)
        ctx.ram_shift(rows, q, b, v0, 1.0, 5, R.RAM_SCAN_F32_TWOSUM)
        torch.cuda.synchronize()
        assert torch.equal(a, b)
