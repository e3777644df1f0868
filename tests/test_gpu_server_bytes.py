"""What a server charges a request against its budget covers what the request
takes on the device, counted by a caller's allocator."""
import ctypes
import threading

import numpy as np
import pytest

from paper_1905_07622_amd import femheat as fh
from paper_1905_07622_amd import workloads as wl
from _util import say

pytestmark = pytest.mark.gpu

ALLOC = ctypes.CFUNCTYPE(ctypes.c_int, ctypes.c_void_p, ctypes.POINTER(ctypes.c_void_p), ctypes.c_size_t,
                         ctypes.c_void_p)
RELEASE = ctypes.CFUNCTYPE(None, ctypes.c_void_p, ctypes.c_void_p, ctypes.c_void_p)


class Allocator(ctypes.Structure):
    _fields_ = [("ctx", ctypes.c_void_p), ("alloc", ALLOC), ("release", RELEASE)]


class Counting:
    """hipMalloc / hipFree, with the bytes held and their peak."""

    def __init__(self):
        self.size, self.held, self.peak, self.calls, self.mu = {}, 0, 0, 0, threading.Lock()
        hip = fh.lib()
        hip.hipFree.argtypes = [ctypes.c_void_p]

        def alloc(_, ptr, n, stream):
            if hip.hipMalloc(ptr, ctypes.c_size_t(n)) != 0:
                return -1
            with self.mu:
                self.size[ptr[0]] = n
                self.held += n
                self.calls += 1
                self.peak = max(self.peak, self.held)
            return 0

        def release(_, p, stream):
            hip.hipFree(p)  # (waits for the stream's work)
            with self.mu:
                self.held -= self.size.pop(p)

        self.struct = Allocator(None, ALLOC(alloc), RELEASE(release))


CASES = [((20, 20, 20), {}), ((99, 99, 99), {}), ((60, 60, 60), dict(precision=fh.FEM_FP32_FP64DOT)),
         ((64, 64, 64), dict(precond=fh.FEM_PRECOND_CHEBYSHEV)), ((40, 40, 40), dict(tile=(16, 8, 16)))]


@pytest.mark.parametrize("dims,opts", CASES)
def test_charged_bytes_cover_the_device_memory(gpu, dims, opts):
    p = wl.random_problem(*dims, seed=2, nsteps=6, dirichlet_value=[0.5] * 6)
    c = Counting()
    so = fh.fem_server_opts()
    so.opts = fh.make_opts(**opts)
    so.opts.allocator = ctypes.addressof(c.struct)
    s = fh.Server.__new__(fh.Server)
    s._pending = {}
    st, s.s = fh.fem_server_create(so)
    assert st == fh.FEM_OK
    with s:
        tickets = [s.submit(p) for _ in range(3)]
        charged = [s.poll(t)["bytes"] for t in tickets]
        for t in tickets:
            assert s.wait(t)[0] == fh.FEM_OK
        info = s.info()
    say(f"  {dims}: {charged[0]} bytes a request, peak {c.peak} allocated, {info['peak_bytes_in_use']} charged")
    # the lane's own records are not a request's: 8 KiB and 16 bytes a brick or block each
    assert c.peak <= info["peak_bytes_in_use"] + 3 * 64 * 1024
    assert c.held == 0


def test_a_launchs_buffers_grow_geometrically(gpu):
    """Runs of 1, 2, ... 300 steps on one handle: the records of a launch grow
    with the steps, but their buffers (pinned, on the device: replacing them
    waits for every stream) are replaced a few times only."""
    p = wl.random_problem(4, 4, 4, seed=2, nsteps=1, rtol=1e-6)
    c = Counting()
    opts = fh.make_opts()
    opts.allocator = ctypes.addressof(c.struct)
    k, r, T = (np.ascontiguousarray(a).ctypes.data_as(fh._dp) for a in (p.k_e, p.rhoc_e, p.T0))
    st, h = fh.fem_heat_create(fh.fem_grid(p.nx, p.ny, p.nz, p.hx, p.hy, p.hz), k, r, None, opts)
    assert st == fh.FEM_OK
    made = c.calls
    for nsteps in range(1, 301):
        assert fh.fem_heat_run(h, T, None, p.dt, p.theta, nsteps, p.rtol, None) == fh.FEM_OK
    grown = c.calls - made
    fh.fem_heat_destroy(h)
    say(f"  {grown} allocations in 300 runs")
    assert grown <= 4 and c.held == 0
