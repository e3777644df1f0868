"""Validation of coefficient arrays in device memory: the same calls are
refused, with the same status and message, as from host arrays (exact), and
the arrays may lie anywhere in an allocation."""
import numpy as np
import pytest

from _util import say
from paper_1905_07622_amd import femheat as fh
from paper_1905_07622_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(1, 1, 1), (11, 10, 9), (33, 32, 31)])
@pytest.mark.parametrize("which,value", [("k_e", -1e-300), ("k_e", np.nan), ("k_e", np.inf), ("rhoc_e", 0.0),
                                         ("rhoc_e", np.nan), ("rhoc_e", -np.inf), ("k_e", -0.0)])
def test_device_arrays_are_refused_as_host_arrays_are(gpu, shape, which, value):
    import torch

    p = wl.random_problem(*shape, seed=3, nsteps=1)
    E = p.k_e.size
    for at in sorted({0, E // 2, E - 1}):
        say(f"{which}[{at}] = {value} on {shape}")
        bad = p.replace(**{which: np.where(np.arange(E) == at, value, getattr(p, which))})

        def on_device(q):  # one element into an allocation that ends with the array
            put = lambda a: torch.tensor(np.concatenate([[np.nan], np.asarray(a)]), device="cuda")[1:]  # noqa: E731
            return q.replace(k_e=put(q.k_e), rhoc_e=put(q.rhoc_e), T0=put(q.T0))

        st, _ = fh.run_batch([p, bad, p], check=False)
        want = fh.fem_last_error(None)
        dst, out = fh.run_batch([on_device(p), on_device(bad), on_device(p)], device_ptrs=True, check=False)
        assert dst == st == (fh.FEM_OK if value == 0 and which == "k_e" else fh.FEM_EINVAL)
        if st != fh.FEM_OK:
            assert fh.fem_last_error(None) == want
