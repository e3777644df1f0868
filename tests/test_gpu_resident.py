"""The resident form (whole steps in one kernel, the grid cut into bricks that
stay on chip) against the oracle, where its cuts can go wrong.

FP64 runs are locked to their own iteration counts and held to 1e-10 of the
oracle, mixed runs to 1e-5 of the FP64 oracle: the gates of the two-kernel
form, whose arithmetic at every node this form shares."""
import threading

import numpy as np
import pytest

from oracle import oracle
from paper_1905_07622_amd import femheat as fh
from paper_1905_07622_amd import workloads as wl
from _util import rel_l2, say

pytestmark = pytest.mark.gpu

GATE64, GATE_MIXED = 1e-10, 1e-5


def problem(dims, seed=5, nsteps=3, **kw):
    """All six faces in play: held at two values, heated, insulated."""
    kw.setdefault("dirichlet_mask", (1 << wl.FACE_XM) | (1 << wl.FACE_ZP))
    kw.setdefault("dirichlet_value", [0.5, 0, 0, 0, 0, -0.25])
    kw.setdefault("flux_mask", 1 << wl.FACE_YP)
    kw.setdefault("flux", [0, 0, 0, 1.0, 0, 0])
    return wl.random_problem(*dims, seed=seed, nsteps=nsteps, rtol=1e-9, **kw)


# one brick; one element; single-file columns and rows; planes that end a brick
# after one plane (c * k + 1 nodes) and exactly at its end; a plate one brick
# high; rows too long for one brick; bricks of the tallest kind on every CU
CUTS = [(1, 1, 1), (6, 5, 2), (1, 1, 39), (300, 1, 1), (1, 200, 2), (16, 16, 17), (16, 16, 18), (20, 7, 44),
        (64, 32, 8), (150, 11, 3), (47, 53, 26), (97, 90, 80)]


@pytest.mark.parametrize("dims", CUTS)
@pytest.mark.parametrize("element", [fh.FEM_ELEM_HEX8, fh.FEM_ELEM_TET6])
def test_cuts_fp64_locked(gpu, dims, element):
    p = problem(dims).replace(element=element)
    with fh.Heat.from_problem(p, replace_every=4) as h:
        out = h.run(p.T0, dt=p.dt, theta=p.theta, nsteps=p.nsteps, rtol=p.rtol, save_every=1)
    ref = oracle.run(p, save_every=1, locked_iters=out["iters"], replace_every=4, nthreads=16)
    errs = [rel_l2(out["T_saved"][n], ref["T_saved"][n]) for n in range(p.nsteps)]
    say(f"  {dims} element {element}: iters {list(out['iters'])} rel L2 {max(errs):.1e}")
    assert out["status"] == fh.FEM_OK and max(errs) <= GATE64
    assert np.all(out["relres"] <= p.rtol)


@pytest.mark.parametrize("dims", CUTS)
def test_cuts_stretched_fp64_locked(gpu, dims):
    p = problem(dims, hx=0.05, hy=0.08, hz=0.03, theta=0.5)
    with fh.Heat.from_problem(p) as h:
        out = h.run(p.T0, dt=p.dt, theta=p.theta, nsteps=p.nsteps, rtol=p.rtol)
    ref = oracle.run(p, locked_iters=out["iters"], nthreads=16)
    assert out["status"] == fh.FEM_OK and rel_l2(out["T_final"], ref["T_final"]) <= GATE64


@pytest.mark.parametrize("degree,dims", [(d, c) for c in CUTS[:-1] for d in (2, 3, 5)] + [(3, (86, 86, 84))])
def test_cuts_chebyshev_locked(gpu, degree, dims):
    """The preconditioner's chain: one exchange (2), one kept vector (3), all
    exchange vectors in use (5); the tallest bricks."""
    p = problem(dims, dt=1e-2, nsteps=1 if dims[2] > 60 else 3)
    with fh.Heat.from_problem(p, replace_every=4, precond=fh.FEM_PRECOND_CHEBYSHEV, cheb_degree=degree) as h:
        out = h.run(p.T0, dt=p.dt, theta=p.theta, nsteps=p.nsteps, rtol=p.rtol, save_every=1)
    ref = oracle.run(p, save_every=1, locked_iters=out["iters"], replace_every=4, nthreads=16,
                     precond=oracle.PRECOND_CHEBYSHEV, cheb_degree=degree)
    errs = [rel_l2(out["T_saved"][n], ref["T_saved"][n]) for n in range(p.nsteps)]
    say(f"  {dims} degree {degree}: iters {list(out['iters'])} rel L2 {max(errs):.1e}")
    assert out["status"] == fh.FEM_OK and max(errs) <= GATE64


@pytest.mark.parametrize("dims", CUTS)
@pytest.mark.parametrize("max_refine,inner_rtol", [(6, 1e-3), (1, 1e-3)])
def test_cuts_mixed(gpu, dims, max_refine, inner_rtol):
    p = problem(dims)
    with fh.Heat.from_problem(p, precision=fh.FEM_FP32_FP64DOT, replace_every=4, max_refine=max_refine,
                              inner_rtol=inner_rtol) as h:
        out = h.run(p.T0, dt=p.dt, theta=p.theta, nsteps=p.nsteps, rtol=p.rtol, check=False)
    assert out["status"] in (fh.FEM_OK, fh.FEM_ENOCONV) and np.all(out["refine_sweeps"] <= max_refine)
    if out["status"] == fh.FEM_OK:
        assert rel_l2(out["T_final"], oracle.run(p, nthreads=16)["T_final"]) <= GATE_MIXED
    else:
        assert max_refine == 1


@pytest.mark.parametrize("precision", [fh.FEM_FP64, fh.FEM_FP32_FP64DOT])
def test_more_bricks_than_compute_units(gpu, precision):
    """A batch whose bricks outnumber the compute units: later simulations wait
    for earlier ones inside the launch.  Kinds and brick heights mixed; every
    member bit for bit as alone."""
    probs = [wl.sphere_proposal(s, n=40, nsteps=3) for s in range(24)]
    probs += [problem((30, 21, 4), seed=9), problem((12, 30, 25), seed=10, hx=0.03, hy=0.05, hz=0.04)]
    st, res = fh.run_batch(probs, precision=precision)
    assert st == fh.FEM_OK
    for k in (0, 11, 23, 24, 25):
        _, alone = fh.run_batch([probs[k]], precision=precision)
        assert np.array_equal(res[k]["T_final"], alone[0]["T_final"]) and np.array_equal(res[k]["iters"], alone[0]["iters"])
    ref = oracle.run(probs[25], **({} if precision else {"locked_iters": res[25]["iters"]}))
    assert rel_l2(res[25]["T_final"], ref["T_final"]) <= (GATE_MIXED if precision else GATE64)


def test_threads_share_the_device(gpu):
    """Four threads, each with its own handle and more bricks than half the
    compute units: every run bit for bit as when it has the device alone."""
    probs = [wl.lognormal_cube(60, seed=s, nsteps=4) for s in range(4)]
    handles = [fh.Heat.from_problem(p) for p in probs]

    def run(k):
        p = probs[k]
        return handles[k].run(p.T0, dt=p.dt, theta=p.theta, nsteps=p.nsteps, rtol=p.rtol)

    alone = [run(k) for k in range(4)]
    got = [[] for _ in range(4)]
    ts = [threading.Thread(target=lambda k=k: got[k].extend(run(k) for _ in range(6))) for k in range(4)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    for k in range(4):
        assert len(got[k]) == 6
        for r in got[k]:
            assert np.array_equal(r["T_final"], alone[k]["T_final"]) and np.array_equal(r["iters"], alone[k]["iters"])
        handles[k].close()


@pytest.mark.parametrize("precision", [fh.FEM_FP64, fh.FEM_FP32_FP64DOT])
def test_blocks_that_do_not_meet(gpu, monkeypatch, precision):
    """The first meeting of a launch made to give up at once (a limit of no
    polls set from the host): nothing has been written then, and the run takes
    the two-kernel form."""
    p = problem((47, 53, 26), nsteps=4)
    monkeypatch.setenv("FEMHEAT_RESIDENT_MEET_LIMIT", "0")
    with fh.Heat.from_problem(p, precision=precision) as h:
        out = h.run(p.T0, dt=p.dt, theta=p.theta, nsteps=p.nsteps, rtol=p.rtol)
    ref = oracle.run(p, **({} if precision else {"locked_iters": out["iters"]}))
    assert out["status"] == fh.FEM_OK
    assert rel_l2(out["T_final"], ref["T_final"]) <= (GATE_MIXED if precision else GATE64)


def test_breakdown_keeps_the_last_good_step(gpu):
    """A step that breaks down (a field that is not finite) ends the run; the
    steps before it stand, as in the two-kernel form."""
    p = problem((20, 18, 15), nsteps=4)
    bad = p.T0.copy()
    bad[1234] = np.inf
    with fh.Heat.from_problem(p) as h:
        out = h.run(bad, dt=p.dt, theta=p.theta, nsteps=p.nsteps, rtol=p.rtol, check=False)
        assert out["status"] == fh.FEM_EBREAKDOWN
        good = h.run(p.T0, dt=p.dt, theta=p.theta, nsteps=p.nsteps, rtol=p.rtol)
    assert good["status"] == fh.FEM_OK
    assert rel_l2(good["T_final"], oracle.run(p, locked_iters=good["iters"])["T_final"]) <= GATE64
