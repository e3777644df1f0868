"""A step that breaks down ends the run with FEM_EBREAKDOWN; the steps before
it stand.  The third step's load is finite in the schedule and overflows on
the grid, so its right-hand side is not finite.  Every form, alone and in a
batch beside a simulation that does not break down."""
import numpy as np
import pytest

from oracle import oracle
from paper_1905_07622_amd import femheat as fh
from paper_1905_07622_amd import workloads as wl
from _util import rel_l2

pytestmark = pytest.mark.gpu

FORMS = [({}, True), (dict(precision=fh.FEM_FP32_FP64DOT), True), (dict(precond=fh.FEM_PRECOND_CHEBYSHEV), True),
         (dict(tile=(0, 0, 12)), False), (dict(tile=(0, 0, 12), precision=fh.FEM_FP32_FP64DOT), False),
         (dict(tile=(0, 0, 12), precond=fh.FEM_PRECOND_CHEBYSHEV), False)]


@pytest.mark.parametrize("opts,resident", FORMS)
@pytest.mark.parametrize("dims", [(6, 5, 2), (20, 18, 15)])
def test_steps_before_a_breakdown_stand(gpu, opts, resident, dims):
    flux = np.zeros(6)
    flux[wl.FACE_ZP] = 1e10
    good = wl.random_problem(*dims, seed=5, nsteps=5, rtol=1e-9)
    p = good.replace(flux_mask=1 << wl.FACE_ZP, flux=flux, flux_schedule=np.array([1e-10, 2e-10, 1e308, 1e-10, 0.0]))
    kw = dict(dt=p.dt, theta=p.theta, nsteps=p.nsteps, rtol=p.rtol, save_every=1)
    with fh.Heat.from_problem(p, **opts) as h:
        h.run(p.T0, **kw, check=False)
        bad = h.run(p.T0, **kw, check=False)
        route = h.route()
        assert bad["status"] == fh.FEM_EBREAKDOWN and "breakdown" in fh.fem_last_error(h.h)
        assert (route["resident_steps"], route["two_kernel_steps"]) == ((2, 0) if resident else (0, 2))
    ref_kw = {} if "precision" in opts else dict(locked_iters=np.asarray(bad["iters"])[:2])
    if "precond" in opts:
        ref_kw.update(precond=oracle.PRECOND_CHEBYSHEV, cheb_degree=3)
    ref = oracle.run(p, nsteps=2, save_every=1, **ref_kw)
    gate = 1e-5 if "precision" in opts else 1e-10
    for n in range(2):
        assert bad["iters"][n] > 0 and rel_l2(bad["T_saved"][n], ref["T_saved"][n]) <= gate
    assert np.array_equal(bad["T_final"], bad["T_saved"][1])
    assert list(bad["iters"][2:]) == [0, 0, 0] and bad["total_iters"] == int(sum(bad["iters"][:2]))
    st, res = fh.run_batch([p, good], save_every=1, check=False, **opts)
    assert st == fh.FEM_EBREAKDOWN and [r["status"] for r in res] == [fh.FEM_EBREAKDOWN, fh.FEM_OK]
    assert rel_l2(res[0]["T_final"], ref["T_saved"][1]) <= gate
    _, alone = fh.run_batch([good], save_every=1, **opts)
    assert np.array_equal(res[1]["T_saved"], alone[0]["T_saved"])
