"""The tile adjoint on uniform runs of the mesh: what a tile in a run takes for
granted changes nothing in the gradient.

* FP64: rows whose nodes are the same in a stretch of equal cells, once a uniform run
  (its cells are the mesh's smallest), once not (two other cells beyond it, one
  smaller and one larger): the gradients there are equal bit for bit.
"""
import numpy as np
import pytest
import torch

from paper_2305_05362_amd import _lib as R

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


def dev(a, dtype=torch.float64):
    return torch.as_tensor(np.ascontiguousarray(a).reshape(-1), dtype=dtype, device=DEV)


@pytest.mark.parametrize("order", [1, 3, 5])
@pytest.mark.parametrize("h", [0.1, 0.7, 1.0 / 3.0])
def test_fp64_gradient_in_a_run(h, order):
    nr, m, k = 4, 2000, 400
    n = m + k
    tail = np.full(k, 2.0 * h)
    other = tail.copy()
    other[[200, 300]] = [0.5 * h, 3.5 * h]
    x = h * np.arange(m + 1.0)
    ea = np.concatenate([x, x[-1] + np.cumsum(tail)])
    eb = np.concatenate([x, x[-1] + np.cumsum(other)])
    eb[-1] = ea[-1]
    rng = np.random.default_rng(2)
    bar = dev(rng.standard_normal((nr, n)))
    v0 = dev(h * np.array([3.37, -2.81, 0.0123, 40.5]))
    got = []
    for e in (ea, eb):
        rows = R.Rows(dev(e), nr, n, None, True)
        paths = R.ram_step_tile_paths(rows, v0, 1.0, order, False).cpu().numpy().reshape(nr, -1)
        assert (paths[:, 1:6] == (R.RAM_TILE_UNIFORM if e is ea else R.RAM_TILE_WINDOW)).all()
        out = torch.empty_like(bar)
        R.ram_step_adjoint(rows, None, None, None, bar, out, v0, 1.0, order)
        got.append(out.cpu().numpy().reshape(nr, n)[:, 320:1400])
    assert np.array_equal(got[0], got[1]), int((got[0] != got[1]).sum())
