"""The launch sequences a call can take, by size, order and capture: the same
results on each."""

import numpy as np
import pytest

from synth import quantize_state

from gpu_helpers import to_device

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pm(gpu):
    import paper_1608_00802_amd as pm_mod
    pm_mod.load_library()
    return pm_mod


def _random(n, npart, seed):
    rng = np.random.default_rng(seed)
    return quantize_state(rng.random((npart, 3)) * n, 0.05 * rng.standard_normal((npart, 3)), n, {})


def test_captured_calls_and_the_spectrum_of_the_deposit(pm, gpu):
    """pm_poisson goes on from the spectrum that pm_deposit left, unless a
    graph may come between: replays of a captured solve, and a solve after
    the replay of a captured force (which uses the spectrum's place), give
    the potential of the deposited density each time."""
    import torch
    n, npart = 64, (1 << 16) + 11
    stream = torch.cuda.Stream(gpu)
    pos, _ = to_device(_random(n, npart, 1), gpu)
    given = [torch.randn(n ** 3, device=gpu) for _ in range(2)]
    acc = torch.empty((3, npart), device=gpu)
    delta, phi, want = (torch.empty(n ** 3, device=gpu) for _ in range(3))
    lp = pm.make_params(n, npart, float(n), hbar_over_m=0.3)
    plain = pm.PMContext(lp, device=gpu)
    plain.deposit(pos, delta)
    plain.poisson(delta.clone(), want)
    torch.cuda.synchronize()

    def check():
        torch.cuda.synchronize()
        assert torch.equal(phi, want)
        phi.zero_()
        torch.cuda.synchronize()

    with torch.cuda.stream(stream):
        ctx = pm.PMContext(lp, device=gpu, stream=stream)
        ctx.deposit(pos)                 # before the capture
        stream.synchronize()
        solve = torch.cuda.CUDAGraph()
        with torch.cuda.graph(solve, stream=stream):
            ctx.poisson(None, phi)
        for _ in range(3):
            solve.replay()
            check()
        ctx.poisson(None, phi)
        check()
        fresh = pm.PMContext(lp, device=gpu, stream=stream)
        force = torch.cuda.CUDAGraph()
        with torch.cuda.graph(force, stream=stream):
            fresh.force(pos, acc, 1.0, *given)
        for _ in range(2):
            fresh.deposit(pos)
            force.replay()
            fresh.poisson(None, phi)
            check()
        torch.cuda.synchronize()
        ctx.close()
        fresh.close()
