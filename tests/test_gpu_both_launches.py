"""Batches of 32768 tiles and more run uniform and searching tiles in two kernels (in
loops of four steps and more as branches of a captured graph), smaller ones in one
launch.  The same tiles' code: the rows that both batches hold come out bit for bit
the same, for every order, with and without residual, for rows that are a multiple
of four cells and rows that are not, in the forward step, the limited step and the
step adjoint with each of its gradients; loops run twice, eager work in between.
"""
import numpy as np
import pytest
import torch

from paper_2305_05362_amd import _lib as R
from paper_2305_05362_amd import workloads as W

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")
FEW, MANY = 16383, 16384                             # rows of two tiles


def dev(a, dtype=torch.float64):
    return torch.as_tensor(np.ascontiguousarray(a).reshape(-1), dtype=dtype, device=DEV)


def inputs(n):
    """A mesh with two uniform runs and a jump between them (both kinds of tile)."""
    rng = np.random.default_rng(n)
    w = np.ones(n)
    w[:40] = 0.25
    e = np.concatenate([[0.0], np.cumsum(w)])
    q = torch.as_tensor(1.0 + 0.2 * rng.standard_normal((MANY, n)), dtype=torch.float32, device=DEV)
    dv = torch.as_tensor(rng.uniform(-1, 1, (MANY, n)), dtype=torch.float32, device=DEV)
    return e, q, dv, dev(rng.uniform(-0.7, 0.7, MANY) * n), 0.1


def rows_of(e, r):
    return R.Rows(dev(e), r, len(e) - 1, None, True)


def part(t, r):
    return None if t is None else t[:r].reshape(-1).contiguous()


def both(run):
    few, many = run(FEW), run(MANY)
    torch.cuda.synchronize()
    for a, b in zip(few, many):
        k = a.numel()
        assert torch.isfinite(a).all()
        assert torch.equal(a, b[:k]), int((a != b[:k]).sum())


@pytest.mark.parametrize("steps", [2, 4])
@pytest.mark.parametrize("with_dv", [True, False])
@pytest.mark.parametrize("order", [1, 3, 5])
@pytest.mark.parametrize("n,scan", [(264, R.RAM_SUM_DIRECT), (268, R.RAM_SCAN_F32_TWOSUM), (265, R.RAM_SUM_DIRECT)])
def test_step(n, scan, order, with_dv, steps):
    e, q0, dv0, v0, dt = inputs(n)

    def run(r):
        rows, out = rows_of(e, r), []
        dv = part(dv0, r) if with_dv else None
        v = v0[:r].contiguous()
        for _ in range(2):
            q = part(q0, r).clone()
            out.append(R.ram_step(rows, q, v, dv, dt, order, steps, scan))
        return out
    both(run)


@pytest.mark.parametrize("steps", [2, 4])
@pytest.mark.parametrize("with_dv", [True, False])
@pytest.mark.parametrize("recon", [R.RAM_RECON_PLM, R.RAM_RECON_PPM])
@pytest.mark.parametrize("n", [264, 265])
def test_limited_step(n, recon, with_dv, steps):
    e, q0, dv0, v0, dt = inputs(n)

    def run(r):
        rows, out = rows_of(e, r), []
        dv = part(dv0, r) if with_dv else None
        v = v0[:r].contiguous()
        for _ in range(2):
            q = part(q0, r).clone()
            out.append(R.ram_step_limited(rows, q, v, dv, dt, recon, steps))
        return out
    both(run)


@pytest.mark.parametrize("with_v0", [True, False])
@pytest.mark.parametrize("with_dv", [True, False])
@pytest.mark.parametrize("order", [1, 3, 5])
def test_step_adjoint(order, with_dv, with_v0):
    n = 264
    e, q0, dv0, v0, dt = inputs(n)
    bar0 = torch.as_tensor(np.random.default_rng(1).standard_normal((MANY, n)), dtype=torch.float32, device=DEV)

    def run(r):
        dv = part(dv0, r) if with_dv else None
        q, bar, out = part(q0, r), part(bar0, r), torch.empty(r * n, dtype=torch.float32, device=DEV)
        dvb = torch.zeros_like(q) if with_dv else None
        v0b = torch.zeros(r, dtype=torch.float64, device=DEV) if with_v0 else None
        R.ram_step_adjoint(rows_of(e, r), q, q if with_dv else None, dv, bar, out, v0[:r].contiguous(), dt,
                           order, dvb, v0b)
        return [t for t in (out, dvb, v0b) if t is not None]
    both(run)
