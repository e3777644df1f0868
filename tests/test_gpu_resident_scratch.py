"""The resident form's scratch takes no device memory of its own where it fits
the field buffer that the form leaves unused."""
import numpy as np
import pytest

from oracle import oracle
from paper_1905_07622_amd import femheat as fh
from paper_1905_07622_amd import workloads as wl
from _util import rel_l2, say

pytestmark = pytest.mark.gpu

MIXED = dict(precision=fh.FEM_FP32_FP64DOT)
CHEB = dict(precond=fh.FEM_PRECOND_CHEBYSHEV)


@pytest.mark.parametrize("n,opts,own", [(100, {}, False), (60, {}, False), (60, MIXED, False), (64, CHEB, True),
                                        (2, {}, True)])
def test_bytes_of_a_resident_simulation(gpu, n, opts, own):
    """Charged as the two-kernel form's, whose tile is named (own: a scratch
    beside the grid's vectors, which are smaller)."""
    p = wl.random_problem(n, n, n, seed=1, nsteps=0)
    charged = []
    for more in ({}, dict(tile=(8, 8, 8))):
        with fh.Server(**opts, **more) as s:
            t = s.submit(p)
            charged.append(s.poll(t)["bytes"])
            s.wait(t)
    say(f"  {n}^3: {charged} bytes")
    assert (charged[0] > charged[1]) == own and charged[0] >= charged[1]


@pytest.mark.parametrize("dims", [(1, 1, 1), (7, 7, 8), (48, 48, 48), (60, 61, 35)])
@pytest.mark.parametrize("opts", [{}, MIXED, CHEB])
def test_replacements_with_the_scratch_in_either_place(gpu, dims, opts):
    """A replacement every third iteration, which puts the direction's halo
    aside in the scratch, alone and as a batch member."""
    p = wl.random_problem(*dims, seed=9, nsteps=3, rtol=1e-9)
    kw = dict(precond=oracle.PRECOND_CHEBYSHEV) if "precond" in opts else {}
    with fh.Heat.from_problem(p, replace_every=3, **opts) as h:
        one = h.run(p.T0, dt=p.dt, theta=p.theta, nsteps=p.nsteps, rtol=p.rtol)
        assert h.route()["resident_steps"] == 3
    st, res = fh.run_batch([p, p], replace_every=3, **opts)
    assert st == fh.FEM_OK and fh.batch_route()["resident_steps"] == 6
    for out in (one, res[0], res[1]):
        lock = {} if "precision" in opts else dict(locked_iters=out["iters"])
        ref = oracle.run(p, replace_every=3, nthreads=8, **lock, **kw)
        err = rel_l2(out["T_final"], ref["T_final"])
        say(f"  {dims} {opts}: {err:.2e}")
        assert err <= (1e-5 if "precision" in opts else 1e-10)
    assert np.array_equal(res[0]["T_final"], res[1]["T_final"])
