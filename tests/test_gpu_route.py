"""Which form takes a run's steps (fem_heat_route): by default the resident
form wherever a grid fits on the chip, the two-kernel form for what names it,
and the two-kernel form from the first step on where a launch's blocks do not
meet.  Fields against the oracle at the gates of both forms (FP64 locked to its
own counts 1e-10, mixed against the FP64 oracle 1e-5)."""
import pytest

from oracle import oracle
from paper_1905_07622_amd import femheat as fh
from paper_1905_07622_amd import workloads as wl
from _util import rel_l2, say

pytestmark = pytest.mark.gpu

GATE64, GATE_MIXED = 1e-10, 1e-5
CHEB = dict(precond=fh.FEM_PRECOND_CHEBYSHEV)
MIXED = dict(precision=fh.FEM_FP32_FP64DOT)

ROUTES = [({}, True), (MIXED, True), (dict(CHEB, cheb_degree=2), True), (dict(CHEB, cheb_degree=5), True),
          (dict(CHEB, cheb_degree=6), False), (dict(tile=(8, 8, 8)), False), (dict(MIXED, tile=(8, 8, 8)), False),
          (dict(one_reduction=True), False), (dict(one_kernel=True), False)]


@pytest.mark.parametrize("opts,resident", ROUTES)
def test_route_of_a_run_and_a_batch(gpu, opts, resident):
    p = wl.random_problem(19, 14, 11, seed=8, nsteps=3, rtol=1e-9)
    with fh.Heat.from_problem(p, **opts) as h:
        assert set(h.route().values()) == {0}
        for nsteps in (3, 2):  # of the last run alone
            h.run(p.T0, dt=p.dt, theta=p.theta, nsteps=nsteps, rtol=p.rtol)
            want = dict(resident_steps=nsteps, two_kernel_steps=0, resident_launches=1, unmet=0) if resident else \
                dict(resident_steps=0, two_kernel_steps=nsteps, resident_launches=0, unmet=0)
            assert h.route() == want
    if "one_kernel" in opts:
        return
    st, _ = fh.run_batch([p, p.replace(nsteps=1), p.replace(nsteps=0)], **opts)
    r = fh.batch_route()
    assert st == fh.FEM_OK and r["unmet"] == 0
    assert (r["resident_steps"], r["two_kernel_steps"]) == ((4, 0) if resident else (0, 4))


@pytest.mark.parametrize("opts", [{}, dict(guess=fh.FEM_GUESS_PREV), MIXED] +
                         [dict(CHEB, cheb_degree=d) for d in (2, 3, 5)])
def test_fallback_runs_where_blocks_do_not_meet(gpu, monkeypatch, opts):
    """A meeting made to give up at once: every step is the two-kernel form's,
    from vectors that the resident launch had prepared for its exchanges."""
    p = wl.random_problem(47, 53, 26, seed=5, nsteps=3, rtol=1e-9, dirichlet_mask=1 << wl.FACE_XM,
                          dirichlet_value=[0.5, 0, 0, 0, 0, 0])
    mixed = "precision" in opts
    kw = dict(guess=oracle.GUESS_PREV) if "guess" in opts else {}
    if "precond" in opts:
        kw = dict(precond=oracle.PRECOND_CHEBYSHEV, cheb_degree=opts["cheb_degree"])
    with fh.Heat.from_problem(p, **opts) as h:
        for limit in (None, "0", None):  # resident, not met, resident again: on the same buffers
            monkeypatch.setenv("FEMHEAT_RESIDENT_MEET_LIMIT", limit) if limit else \
                monkeypatch.delenv("FEMHEAT_RESIDENT_MEET_LIMIT", raising=False)
            out = h.run(p.T0, dt=p.dt, theta=p.theta, nsteps=p.nsteps, rtol=p.rtol)
            r = h.route()
            ref = oracle.run(p, **(kw if mixed else dict(kw, locked_iters=out["iters"])), nthreads=16)
            err = rel_l2(out["T_final"], ref["T_final"])
            say(f"  limit {limit}: {r} rel L2 {err:.1e}")
            assert out["status"] == fh.FEM_OK and err <= (GATE_MIXED if mixed else GATE64)
            assert (r["resident_steps"], r["two_kernel_steps"], r["unmet"]) == \
                ((0, p.nsteps, 1) if limit else (p.nsteps, 0, 0))


def test_fallback_of_batch_members(gpu, monkeypatch):
    probs = [wl.sphere_proposal(s, n=30, nsteps=3) for s in range(4)]
    monkeypatch.setenv("FEMHEAT_RESIDENT_MEET_LIMIT", "0")
    st, res = fh.run_batch(probs)
    r = fh.batch_route()
    say(f"  {r}")
    assert st == fh.FEM_OK and (r["resident_steps"], r["two_kernel_steps"], r["unmet"]) == (0, 12, 4)
    for p, o in zip(probs, res):
        assert rel_l2(o["T_final"], oracle.run(p, locked_iters=o["iters"])["T_final"]) <= GATE64
