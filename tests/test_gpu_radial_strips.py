"""The radial step around its strips' lengths: rows that end a strip of four or
eight rows, one less and one more, and on either side of the numbers of strips
where they go from four rows to eight (1024 workgroups) and, in FP32, on to
sixteen (4096).  Against the oracle at
the radial tests' bars (FP64 1e-12 relative L1, FP32 1e-6 on FP32 inputs).
"""
import numpy as np
import pytest
import torch

import oracle
from parity import rel_l1
from paper_2305_05362_amd import _lib as R
from paper_2305_05362_amd import workloads as W

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


@pytest.mark.parametrize("dtype,bar", [(torch.float64, 1e-12), (torch.float32, 1e-6)])
@pytest.mark.parametrize("n_r", [3, 4, 5, 8, 9, 8183, 8184, 8185, 8192, 8193, 32760, 32761])
def test_strips(n_r, dtype, bar):
    wl = W.small_polar(n_r, 64, 2)
    u = W.radial_velocity(wl, 2, amp=0.05)
    dt = min(wl.dt, W.radial_cfl_dt(wl.meta["r_edges"], u, 0.5))
    q = np.asarray(wl.q0, dtype=np.float32).astype(np.float64)
    u = np.asarray(u, dtype=np.float32).astype(np.float64)

    def dev(a, t=dtype):
        return torch.as_tensor(np.ascontiguousarray(a).reshape(-1), dtype=t, device=DEV)

    out = torch.empty(wl.n_cells, dtype=dtype, device=DEV)
    R.ram_radial_step(R.Rows.from_workload(wl, DEV), dev(q), out,
                      dev(wl.meta["r_edges"], torch.float64), dev(u), dt)
    torch.cuda.synchronize()
    want = oracle.radial(wl.meta["r_edges"], q, u, dt)
    assert rel_l1(out.cpu().numpy(), np.asarray(want).reshape(-1)) <= bar
