"""Resident launches on a device that they do not have to themselves: blocks
that wait for compute units, and work that waits for theirs."""
import ctypes
import threading
import time

import numpy as np
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


def same_bits(a, b):
    for key in ("T_final", "T_saved", "traces", "iters", "relres", "refine_sweeps"):
        assert (a[key] is None) == (b[key] is None)
        assert a[key] is None or np.array_equal(a[key], b[key]), key


@pytest.mark.parametrize("dims", [(6, 5, 2), (16, 16, 17), (47, 53, 26)])
@pytest.mark.parametrize("opts", [{}, dict(precision=fh.FEM_FP32_FP64DOT), dict(precond=fh.FEM_PRECOND_CHEBYSHEV)])
def test_short_launches_change_no_bits(gpu, monkeypatch, opts, dims):
    """A launch that may hold its compute units for no time at all (set from
    the host) ends after one step: as many launches as steps, and the same
    fields, counts and traces as from one launch.  One brick and many; fields
    saved and not."""
    p = wl.random_problem(*dims, seed=21, nsteps=7, rtol=1e-9)
    xyz = np.random.default_rng(4).uniform(0, 1, (5, 3)) * [p.nx * p.hx, p.ny * p.hy, p.nz * p.hz]
    for save_every in (0, 3):
        kw = dict(dt=p.dt, theta=p.theta, nsteps=p.nsteps, rtol=p.rtol, sensors=xyz, save_every=save_every)
        with fh.Heat.from_problem(p, **opts) as h:
            one = h.run(p.T0, **kw)
            assert h.route()["resident_launches"] == (3 if save_every else 1)
            monkeypatch.setenv("FEMHEAT_RESIDENT_LAUNCH_MS", "0")
            each = h.run(p.T0, **kw)
            r = h.route()
            monkeypatch.delenv("FEMHEAT_RESIDENT_LAUNCH_MS")
        assert (r["resident_launches"], r["resident_steps"]) == (7, 7)
        same_bits(each, one)
    monkeypatch.setenv("FEMHEAT_RESIDENT_LAUNCH_MS", "0")
    st, res = fh.run_batch([p, p.replace(nsteps=2)], **opts)
    assert st == fh.FEM_OK and fh.batch_route()["resident_steps"] == 9 and fh.batch_route()["resident_launches"] == 9  # in turn
    monkeypatch.delenv("FEMHEAT_RESIDENT_LAUNCH_MS")
    _, whole = fh.run_batch([p, p.replace(nsteps=2)], **opts)
    for a, b in zip(res, whole):
        same_bits(a, b)


def stiff(n, nsteps):
    """Steps that never converge: every one takes max_iter iterations."""
    return wl.lognormal_cube(n, seed=3, nsteps=nsteps).replace(rtol=1e-30)


def test_a_long_run_gives_the_device_back_in_between(gpu):
    """128 steps of 300 iterations (about 2 ms each) are more than one launch
    holds the device for (100 ms)."""
    p = stiff(64, 128)
    with fh.Heat.from_problem(p, max_iter=300) as h:
        out = h.run(p.T0, dt=p.dt, theta=p.theta, nsteps=p.nsteps, rtol=p.rtol, check=False)
        r = h.route()
    say(f"  {out['device_ms']:.0f} ms in {r['resident_launches']} launches")
    assert out["status"] == fh.FEM_ENOCONV and r["resident_steps"] == 128
    assert max(2, out["device_ms"] / 110) <= r["resident_launches"] <= out["device_ms"] / 100 + 1


def test_a_stiff_request_gives_the_device_back_after_each_step(gpu):
    """Steps of 2 ms and more are as long as a server's launch may be: one per
    epoch, so that requests of other sizes get their turn in between."""
    p = stiff(80, 8)
    with fh.Server(max_iter=400) as s:
        st, _, _ = s.wait(s.submit(p))
        assert st == fh.FEM_ENOCONV
        assert s.info()["epochs"] == 8  # (two of four steps each without the bound)


def test_one_kernel_iterations_beside_resident_runs(gpu, monkeypatch):
    """Runs with FEM_ONE_KERNEL while other threads' resident launches take
    nearly every compute unit for 100 ms at a time: the grid barrier, whose
    wait is made short (about 10 ms), never waits for them."""
    busy = stiff(96, 40)
    p = wl.lognormal_cube(48, seed=6, nsteps=20)
    stop = threading.Event()
    statuses = []

    def keep_busy():
        with fh.Heat.from_problem(busy, max_iter=400) as h:
            while not stop.is_set():
                statuses.append(h.run(busy.T0, dt=busy.dt, theta=busy.theta, nsteps=busy.nsteps, rtol=busy.rtol,
                                      check=False)["status"])

    with fh.Heat.from_problem(p, one_kernel=True, timing=True) as h:
        kw = dict(dt=p.dt, theta=p.theta, nsteps=p.nsteps, rtol=p.rtol)
        alone = h.run(p.T0, **kw)
        assert h.stats()["one_kernel_launches"] > 0
        monkeypatch.setenv("FEMHEAT_BARRIER_SPIN_LIMIT", "20000")
        t = threading.Thread(target=keep_busy)
        t.start()
        try:
            time.sleep(0.3)
            beside = [h.run(p.T0, **kw) for _ in range(3)]
        finally:
            stop.set()
            t.join()
    assert set(statuses) == {fh.FEM_ENOCONV}
    for out in beside:
        same_bits(out, alone)


@pytest.mark.parametrize("opts", [{}, dict(precision=fh.FEM_FP32_FP64DOT)])
def test_more_simulations_than_the_preparing_grid_has_rows(gpu, opts):
    """1100 small simulations of several bricks in one launch (the kernel that
    prepares a launch takes 1024 at a time): each bit for bit as alone."""
    probs = [wl.random_problem(1, 1, 39, seed=s % 50, nsteps=2, rtol=1e-9) for s in range(1100)]
    st, res = fh.run_batch(probs, **opts)
    r = fh.batch_route()
    assert st == fh.FEM_OK and (r["resident_steps"], r["unmet"]) == (2200, 0)
    for s in range(50):
        _, alone = fh.run_batch([probs[s]], **opts)
        for k in range(s, 1100, 50):
            same_bits(res[k], alone[0])
