"""The two-kernel form under the tests of runs, batches, servers and
preconditioners.

Those tests name no tile, and their grids fit on the chip, so they run in the
resident form.  The two-kernel form serves the grids that do not fit, named
tiles, Chebyshev degrees above 5 and launches whose blocks do not meet: here
the same tests run with the z-chunk of the gather's tile named (nothing else
of the tile rule changes), and every run is checked to have taken it.  So the
lockstep batches with their compaction and concurrent groups, the early
refinement sweeps, the next step behind a decide and the preconditioner's
chain of gathers stay under test, at the gates that those tests state."""
import itertools

import numpy as np
import pytest

import test_gpu_batch
import test_gpu_cheb
import test_gpu_mixed
import test_gpu_run
import test_gpu_server
import test_gpu_tet
from oracle import oracle
from paper_1905_07622_amd import femheat as fh
from paper_1905_07622_amd import workloads as wl
from _util import rel_l2, say

pytestmark = pytest.mark.gpu

TILE = (0, 0, 12)


def cases(module, *names):
    """(function, arguments) of every parametrisation of a module's tests."""
    for name in names:
        fn = getattr(module, name)
        sets = []
        for m in getattr(fn, "pytestmark", []):
            if m.name == "parametrize":
                keys = [k.strip() for k in m.args[0].split(",")]
                sets.append([dict(zip(keys, v if len(keys) > 1 else (v,))) for v in m.args[1]])
        for k, combo in enumerate(itertools.product(*sets)):
            yield pytest.param(fn, {a: v for c in combo for a, v in c.items()}, id=f"{module.__name__}-{name[5:]}-{k}")


CASES = [
    *cases(test_gpu_batch, *[n for n in dir(test_gpu_batch) if n.startswith("test_")]),
    *cases(test_gpu_run, "test_sphere_cube_full_run", "test_small_runs_locked_parity",
           "test_sensor_traces_and_flux_schedule", "test_resume_equals_uninterrupted",
           "test_deterministic_and_edge_cases", "test_zero_rhs_gives_zero_field", "test_full_size_lognormal_first_steps",
           "test_timing_changes_nothing_and_samples"),
    *cases(test_gpu_mixed, "test_mixed_sphere_cube", "test_mixed_lognormal_and_flux", "test_mixed_slab_sensors",
           "test_mixed_full_size_slab_first_steps"),
    *cases(test_gpu_cheb, "test_cheb_runs_locked_parity", "test_cheb_lognormal_fewer_iterations_same_field",
           "test_cheb_batch_alone_equals_mix"),
    *cases(test_gpu_tet, "test_tet_runs_locked_parity", "test_tet_mixed_and_batch"),
    *cases(test_gpu_server, "test_continuous_batching_results_equal_alone_and_oracle", "test_cancel_queued_and_running",
           "test_one_slot_admits_in_arrival_order_across_classes", "test_mixed_precision_server"),
]


@pytest.fixture
def named_tile(monkeypatch):
    """Names TILE wherever no tile is given; counts the steps of each form."""
    seen = {"resident_steps": 0, "two_kernel_steps": 0, "unmet": 0}

    def count(route):
        for k in seen:
            seen[k] += route[k]

    def with_tile(call):
        def inner(*a, **kw):
            kw.setdefault("tile", TILE)
            return call(*a, **kw)
        return inner

    batch, run = fh.run_batch, fh.Heat.run

    def counted_batch(*a, **kw):
        out = batch(*a, **kw)
        count(fh.batch_route())
        return out

    def counted_run(self, *a, **kw):
        out = run(self, *a, **kw)
        count(self.route())
        return out

    monkeypatch.setattr(fh, "run_batch", with_tile(counted_batch))
    monkeypatch.setattr(fh.Heat, "run", counted_run)
    monkeypatch.setattr(fh.Heat, "__init__", with_tile(fh.Heat.__init__))
    monkeypatch.setattr(fh.Server, "__init__", with_tile(fh.Server.__init__))
    return seen


@pytest.mark.parametrize("test,kw", CASES)
def test_in_the_two_kernel_form(gpu, named_tile, test, kw):
    test(gpu, **kw)
    say(f"  {named_tile}")
    assert named_tile["resident_steps"] == 0 and named_tile["unmet"] == 0
    assert named_tile["two_kernel_steps"] > 0 or test.__module__ == "test_gpu_server"


@pytest.mark.parametrize("degree", [6, 7, 8])
@pytest.mark.parametrize("dims", [(13, 9, 11), (40, 33, 18)])
def test_long_preconditioner_chains(gpu, degree, dims):
    """Degrees that have no resident form: alone and in a batch (bit for bit
    the same in a mix), against the oracle locked to their counts."""
    probs = [wl.random_problem(*dims, seed=81 + k, nsteps=4 - k, dt=1e-2, rtol=1e-10, k_range=(0.01, 100.0),
                               dirichlet_mask=1 << wl.FACE_XP, dirichlet_value=[0, 1.5, 0, 0, 0, 0]) for k in range(3)]
    out, ref = test_gpu_cheb.run_both(probs[0], degree, heat_kw=dict(replace_every=3))
    assert out["status"] == 0
    assert max(rel_l2(out["T_saved"][n], ref["T_saved"][n]) for n in range(probs[0].nsteps)) <= 1e-10
    kw = dict(precond=fh.FEM_PRECOND_CHEBYSHEV, cheb_degree=degree)
    st, mix = fh.run_batch(probs, **kw)
    assert st == fh.FEM_OK and fh.batch_route()["two_kernel_steps"] == 4 + 3 + 2
    for p, r in zip(probs, mix):
        _, alone = fh.run_batch([p], **kw)
        assert np.array_equal(alone[0]["T_final"], r["T_final"]) and np.array_equal(alone[0]["iters"], r["iters"])
        ref = oracle.run(p, locked_iters=r["iters"], precond=oracle.PRECOND_CHEBYSHEV, cheb_degree=degree)
        assert rel_l2(r["T_final"], ref["T_final"]) <= 1e-10


def test_tuned_tiles_in_runs(gpu, tmp_path):
    """Tiles from the autotuner's cache, alone and as batch members, in runs
    that use the gather."""
    p = wl.lognormal_cube(30, seed=5, nsteps=3).replace(dt=2e-3)
    kw = dict(precond=fh.FEM_PRECOND_CHEBYSHEV, cheb_degree=6, tune_cache=str(tmp_path / "tune.json"))
    okw = dict(precond=oracle.PRECOND_CHEBYSHEV, cheb_degree=6)
    with fh.Heat.from_problem(p, **kw) as h:
        best = h.tune(dt=p.dt, theta=p.theta)
        assert h.tune(dt=p.dt, theta=p.theta, batch=True)["recorded"] == 1
        runs = [h.run(p.T0, dt=p.dt, theta=p.theta, nsteps=p.nsteps, rtol=p.rtol)]
    with fh.Heat.from_problem(p, **kw) as h:
        assert [h.stats()[k] for k in ("tile_x", "tile_y", "tile_z")] == [best[k] for k in ("tile_x", "tile_y", "tile_z")]
        runs.append(h.run(p.T0, dt=p.dt, theta=p.theta, nsteps=p.nsteps, rtol=p.rtol))
        assert h.route()["two_kernel_steps"] == p.nsteps
    assert np.array_equal(runs[0]["T_final"], runs[1]["T_final"])
    st, res = fh.run_batch([p, p.replace(nsteps=2)], **kw)
    assert st == fh.FEM_OK and fh.batch_route()["two_kernel_steps"] == 5
    for out in (runs[1], res[0]):
        ref = oracle.run(p, locked_iters=out["iters"], **okw)
        assert rel_l2(out["T_final"], ref["T_final"]) <= 1e-10
