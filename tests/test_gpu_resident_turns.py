"""Simulations of a launch that wait for their turn through several launches
take the same steps, bit for bit, as those that run in the first."""
import numpy as np
import pytest

from paper_1905_07622_amd import femheat as fh
from paper_1905_07622_amd import workloads as wl
from _util import say

pytestmark = pytest.mark.gpu

MIXED = dict(precision=fh.FEM_FP32_FP64DOT)
CHEB = dict(precond=fh.FEM_PRECOND_CHEBYSHEV)


@pytest.mark.parametrize("opts", [{}, MIXED, CHEB])
def test_turns_change_no_bits(gpu, monkeypatch, opts):
    """Launches that are over at once (set from the host): each takes one step
    of one simulation, the others wait with the vectors that the first launch
    prepared.  Cuts of one brick and of many, and of each height."""
    dims = [(6, 5, 2), (7, 8, 8), (33, 20, 4), (40, 37, 17), (47, 53, 26), (40, 37, 17), (6, 5, 2)]
    probs = [wl.random_problem(*d, seed=30 + k, nsteps=1 + k % 3, rtol=1e-9, dirichlet_value=[0.25] * 6)
             for k, d in enumerate(dims)]
    _, whole = fh.run_batch(probs, replace_every=7, **opts)
    assert fh.batch_route()["resident_steps"] == sum(p.nsteps for p in probs)
    monkeypatch.setenv("FEMHEAT_RESIDENT_LAUNCH_MS", "0")
    st, turns = fh.run_batch(probs, replace_every=7, **opts)
    r = fh.batch_route()
    assert st == fh.FEM_OK and (r["resident_steps"], r["unmet"]) == (sum(p.nsteps for p in probs), 0)
    for a, b in zip(turns, whole):
        for key in ("T_final", "iters", "relres"):
            assert np.array_equal(a[key], b[key]), key


def test_launches_of_a_pass_take_turns(gpu):
    """Requests of one size class that run in two kernels (boxes, and cubic
    elements), steps as long as a launch may last: the ones do not wait until
    the others are done.  In turns, 8 short requests take one step each in every
    second epoch; one step of one of them in each epoch would be 64 epochs."""
    short = [wl.random_problem(20, 20, 20, seed=s, nsteps=8, rtol=1e-30) for s in range(8)]
    long = [p.replace(hz=1.5 * p.hz, nsteps=60) for p in short[:4]]
    with fh.Server(max_iter=600) as s:
        running = [s.submit(p) for p in long]
        for t in [s.submit(p) for p in short]:
            assert s.wait(t)[0] == fh.FEM_ENOCONV
        epochs = s.info()["epochs"]
        assert any(s.poll(t)["state"] == fh.FEM_REQ_RUNNING for t in running)
    say(f"  {epochs} epochs")
    assert epochs <= 32
