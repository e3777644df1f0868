"""The benchmark names the form that the library says it took (no GPU)."""
import os
import sys

import pytest

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
import bench  # noqa: E402


@pytest.mark.parametrize("resident,other,otherwise,form", [
    (200, 0, "two-kernel", "resident"), (0, 200, "two-kernel", "two-kernel"), (0, 200, "one-kernel", "one-kernel"),
    (128, 72, "two-kernel", "resident, then two-kernel"), (0, 0, "two-kernel", "two-kernel")])
def test_form_taken(resident, other, otherwise, form):
    route = dict(resident_steps=resident, two_kernel_steps=other, resident_launches=1, unmet=0)
    assert bench.form_taken(route, otherwise) == form


def test_resident_roofline_counts_the_whole_iteration():
    """Operations against the time that an iteration takes of the run, not the
    sampled part of it."""
    N = 1000000
    r = bench.resident_roofline(N, 8, 14.0, {"gather": 6.5e-3, "update": 4.5e-3})
    assert r["achieved"] == round(126 * N / 14.0e-6 / 1e12, 2) and r["iteration_us"] == 14.0
    assert r["frac"] == pytest.approx(126 * N / 14.0e-6 / 1e12 / 78.6, abs=1e-4)
    assert r["halves_us"] == {"gather": 6.5, "update": 4.5}
