"""Grids whose node count overflows 32 bits are refused before any array is
read, whatever the pointers' kind (CPU only: nothing reaches a device)."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CALL = """
import ctypes, sys
import numpy as np
sys.path.insert(0, {root!r})
from paper_1905_07622_amd import femheat as fh
one = np.ones(8).ctypes.data_as(fh._dp)
grid = fh.fem_grid({nx}, {ny}, {nz}, 1.0, 1.0, 1.0)
opts = fh.make_opts(device_ptrs={dev})
if {batch}:
    req = fh.fem_request()
    req.grid, req.k_e, req.rhoc_e, req.T0, req.dt, req.theta, req.rtol, req.nsteps = grid, one, one, one, 1.0, 1.0, 1.0, 1
    st = fh.fem_heat_run_batch(ctypes.pointer(req), 1, opts, None)
else:
    st, _ = fh.fem_heat_create(grid, one, one, None, opts)
assert st == fh.FEM_EINVAL and "too large" in fh.fem_last_error(None), (st, fh.fem_last_error(None))
"""

MAX = 2**31 - 1


@pytest.mark.parametrize("n", [(MAX, 1, 1), (1, MAX, 1), (MAX, 2, MAX), (MAX, MAX, MAX), (MAX - 1, 1, 1)])
@pytest.mark.parametrize("dev", [False, True])
@pytest.mark.parametrize("batch", [False, True])
def test_overflowing_grids_are_refused(n, dev, batch):
    code = CALL.format(root=ROOT, nx=n[0], ny=n[1], nz=n[2], dev=dev, batch=batch)
    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, (r.returncode, r.stderr[-1500:])
