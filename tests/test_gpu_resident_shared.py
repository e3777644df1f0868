"""Resident launches on a device that they do not have to themselves: blocks
that wait for compute units, and work that waits for theirs."""
import ctypes
import time

import pytest

from oracle import oracle
from paper_1905_07622_amd import femheat as fh
from paper_1905_07622_amd import workloads as wl
from _util import rel_l2, say

pytestmark = pytest.mark.gpu

GATE64 = 1e-10


def test_members_wait_while_earlier_ones_run(gpu, monkeypatch):
    """Bricks of a batch outnumber the compute units several times over, and
    every member runs for much longer than a meeting may take (a limit of 300
    polls, 0.2 ms, set from the host): the time that an earlier member runs
    does not count, and all members stay resident."""
    probs = [wl.sphere_proposal(s, n=48, nsteps=4) for s in range(32)]
    monkeypatch.setenv("FEMHEAT_RESIDENT_MEET_LIMIT", "300")
    st, res = fh.run_batch(probs)
    r = fh.batch_route()
    say(f"  {r}")
    assert st == fh.FEM_OK and (r["resident_steps"], r["unmet"]) == (32 * 4, 0)
    for k in (0, 31):
        assert rel_l2(res[k]["T_final"], oracle.run(probs[k], locked_iters=res[k]["iters"])["T_final"]) <= GATE64


@pytest.mark.parametrize("members", [1, 3])
def test_a_launch_that_cannot_have_its_compute_units_gives_up_soon(gpu, members):
    """A stream that may use a quarter of the compute units: no member can
    meet.  Each gives up after 20 ms, also in a launch with more blocks than
    the device has compute units, and runs in the two-kernel form."""
    probs = [wl.random_problem(97, 90, 40, seed=s, nsteps=2, rtol=1e-9) for s in range(members)]
    hip = fh.lib()  # (its HIP runtime)
    mask = (ctypes.c_uint32 * 2)(0xFFFFFFFF, 0xFFFFFFFF)
    stream = ctypes.c_void_p()
    assert hip.hipExtStreamCreateWithCUMask(ctypes.byref(stream), 2, mask) == 0
    try:
        t0 = time.perf_counter()
        st, res = fh.run_batch(probs, stream=stream.value)
        secs = time.perf_counter() - t0
    finally:
        assert hip.hipStreamSynchronize(stream) == 0 and hip.hipStreamDestroy(stream) == 0
    r = fh.batch_route()
    say(f"  {members} members: {r} in {secs:.2f} s")
    assert st == fh.FEM_OK and (r["two_kernel_steps"], r["unmet"]) == (2 * members, members)
    assert secs < 5.0
    for p, o in zip(probs, res):
        assert rel_l2(o["T_final"], oracle.run(p, locked_iters=o["iters"], nthreads=8)["T_final"]) <= GATE64
