"""The tables of a shared mesh: a host check of where they lie (csrc/ram_mesh_layout.h,
built with g++, no HIP headers), and ram_shift_noalloc on the largest meshes its
static buffer holds (16 MiB at 552 bytes a cell), which it took for too large while
the tables' size counted two that were no longer there."""
import os
import shutil
import subprocess

import numpy as np
import pytest
import torch

from paper_2305_05362_amd import _lib as R

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2305_05362_amd", "csrc")
SRC = os.path.join(ROOT, "tests", "host", "mesh_layout_check.cpp")


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_layout(tmp_path):
    exe = str(tmp_path / "mesh_layout_check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", CSRC, SRC, "-o", exe], check=True)
    out = subprocess.run([exe], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout + out.stderr
    assert "all checks passed" in out.stdout


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,scan", [(torch.float64, R.RAM_SCAN_F64), (torch.float32, R.RAM_SUM_DIRECT)])
def test_noalloc_on_a_mesh_that_fits(dtype, scan):
    n, nr, dev = 29000, 2, torch.device("cuda:0")
    rng = np.random.default_rng(5)
    e = np.concatenate([[0.0], np.cumsum(8.0 ** rng.random(n))])
    rows = R.Rows(torch.as_tensor(e, device=dev), nr, n, None, True)
    q = torch.as_tensor(rng.uniform(0.5, 2.0, nr * n), dtype=dtype, device=dev)
    v0 = torch.as_tensor(np.array([0.3, -0.7]) * e[-1], device=dev)
    ctx = R.context(0)
    a, b = torch.full_like(q, float("nan")), torch.full_like(q, float("nan"))
    ctx.set_schedule(4)
    try:
        ctx.ram_shift_noalloc(rows, q, a, v0, 1.0, 5, scan)
        ctx.ram_shift(rows, q, b, v0, 1.0, 5, scan)
        torch.cuda.synchronize()
    finally:
        ctx.set_schedule(0)
    assert torch.equal(a, b)
