"""Creating a handle and running it wait for no other stream's work."""
import pytest

from paper_1905_07622_amd import femheat as fh
from paper_1905_07622_amd import workloads as wl
from _util import say

pytestmark = pytest.mark.gpu


def keep_busy(torch, s, ms):
    """A kernel of one block on s that lasts about ms; an event behind it."""
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
    cycles = 2_000_000
    with torch.cuda.stream(s):
        torch.cuda._sleep(1000)
        ev[0].record()
        torch.cuda._sleep(cycles)
        ev[1].record()
    torch.cuda.synchronize()
    done = torch.cuda.Event()
    with torch.cuda.stream(s):
        torch.cuda._sleep(int(cycles * ms / ev[0].elapsed_time(ev[1])))
        done.record()
    return done


def stream_beside(torch, mine):
    """A stream that shares its hardware queue (a process has four) neither
    with the default stream nor with `mine`."""
    x = torch.zeros(64, device="cuda")
    for _ in range(8):
        s = torch.cuda.Stream()
        done = keep_busy(torch, s, 100)
        for other in (torch.cuda.default_stream(), mine):
            with torch.cuda.stream(other):
                x.add_(1.0)
            other.synchronize()
        beside = not done.query()
        torch.cuda.synchronize()
        if beside:
            return s
    raise AssertionError("no stream beside the default stream")


@pytest.mark.parametrize("n", [4, 20])
@pytest.mark.parametrize("dev", [False, True])
def test_create_and_run_beside_other_work(gpu, dev, n):
    import torch

    p = wl.random_problem(n, n, n, seed=1, nsteps=2)
    if dev:
        put = lambda a: torch.tensor(a, device="cuda")  # noqa: E731
        p = p.replace(k_e=put(p.k_e), rhoc_e=put(p.rhoc_e), T0=put(p.T0))
    mine = torch.cuda.Stream()
    s = stream_beside(torch, mine)
    opts = dict(device_ptrs=dev, stream=mine.cuda_stream)
    with fh.Heat.from_problem(p, **opts) as h:  # (the first use of everything)
        h.run(p.T0, dt=p.dt, theta=p.theta, nsteps=p.nsteps, rtol=p.rtol)
    done = keep_busy(torch, s, 600)
    h = fh.Heat.from_problem(p, **opts)
    created_beside = not done.query()
    for nsteps in (1, 40):
        h.run(p.T0, dt=p.dt, theta=p.theta, nsteps=nsteps, rtol=p.rtol)
    ran_beside = not done.query()
    torch.cuda.synchronize()
    h.close()
    say(f"  created beside: {created_beside}, ran beside: {ran_beside}")
    assert created_beside and ran_beside
