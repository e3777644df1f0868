"""Host memory that runs out while a call looks its requests over ends in
FEM_ENOMEM, not in an exception that leaves the library (CPU only: the calls
stop before they read an array or reach a device)."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# 256 MB of address space left, requests whose own tables take 512 MB
CALL = """
import ctypes, resource, sys
import numpy as np
sys.path.insert(0, {root!r})
from paper_1905_07622_amd import femheat as fh
one = np.ones(8).ctypes.data_as(fh._dp)
opts = fh.make_opts(device_ptrs={dev})
grid = fh.fem_grid(2**26, 1, 1, 1.0, 1.0, 1.0)
req = fh.fem_request()
fh.lib()
used = int(open("/proc/self/statm").read().split()[0]) * resource.getpagesize()
resource.setrlimit(resource.RLIMIT_AS, (used + (256 << 20), -1))
if {batch}:
    st = fh.fem_heat_run_batch(ctypes.pointer(req), 2**27, opts, None)
else:
    st, _ = fh.fem_heat_create(grid, one, one, None, opts)
assert st == fh.FEM_ENOMEM and "host" in fh.fem_last_error(None), (st, fh.fem_last_error(None))
"""


@pytest.mark.parametrize("batch,dev", [(True, False), (True, True), (False, False)])
def test_no_exception_leaves_the_library(batch, dev):
    code = CALL.format(root=ROOT, batch=batch, dev=dev)
    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, (r.returncode, r.stderr[-1500:])
