"""Simulations of a launch that wait for their turn through several launches
take the same steps, bit for bit, as those that run in the first."""
import numpy as np
import pytest

from paper_1905_07622_amd import femheat as fh
from paper_1905_07622_amd import workloads as wl

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
