"""Single kernels and dispatch branches at the sizes where they can go wrong,
against the FP64 oracle or against the general path of the same call."""

import numpy as np
import pytest

import oracle
from synth import quantize_state

from gpu_helpers import to_device

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pm(gpu):
    import paper_1608_00802_amd as pm_mod
    pm_mod.load_library()
    return pm_mod


def _state(n, npart, seed, clumps=True):
    """Random particles, with clumps most of them in a few dense objects (one
    of them across the box corner) over a sparse background."""
    rng = np.random.default_rng(seed)
    pos = rng.random((npart, 3)) * n
    if clumps:
        centres = np.concatenate([np.zeros((1, 3)), rng.random((3, 3)) * n])
        pick = rng.random(npart) < 0.8
        k = rng.integers(0, 4, npart)
        pos[pick] = (centres[k] + 1.2 * rng.standard_normal((npart, 3)))[pick]
    return quantize_state(pos % n, 0.05 * rng.standard_normal((npart, 3)), n, {})


@pytest.mark.parametrize("n,npart", [(16, 1), (16, 3001), (16, 20001), (32, 32 ** 3),
                                     (64, 40 ** 3 + 17)])
def test_float_tiled_deposit(pm, gpu, n, npart):
    """Windows summed in FP64: a weight takes two roundings (1 - f is exact),
    a window's sum one, and adding at most eight windows to a node one each:
    11 half-ulps, below 2^-20 of the node's value."""
    import torch
    st = _state(n, npart, seed=n + npart)
    ctx = pm.PMContext(pm.make_params(n, npart, float(n), precision=pm.PM_FP32), device=gpu)
    pos, vel = to_device(st, gpu, fp32_positions=True)
    ctx.sort(pos, vel)
    ctx.deposit(pos)
    torch.cuda.synchronize()
    acc = ctx.workspace[: 4 * n ** 3].view(torch.float32).cpu().numpy().astype(np.float64)
    x = pos.cpu().numpy().T.astype(np.float64)
    ref = oracle.deposit(x, oracle.Params(n=n, box=float(n), S=1.0, hbar_m=0.0)).ravel()
    ref *= npart / n ** 3
    assert np.all(np.abs(acc - ref) <= 2.0 ** -20 * ref + 1e-30)


def _rows(pos, vel):
    """Order-free view of a state: its rows (x, y, z, vx, vy, vz) sorted."""
    import torch
    a = torch.cat([pos.view(torch.int32), vel.view(torch.int32)]).cpu().numpy()
    return a[:, np.lexsort(a[::-1])]


@pytest.mark.parametrize("n,npart,move", [(16, 1, 0.3), (16, 513, 0.3), (16, 8193, 2.5),
                                          (32, 20001, 0.3), (64, 70001, 2.5)])
def test_tiled_step_equals_direct_step(pm, gpu, n, npart, move):
    """The two-phase gather-deposit against the direct kernels, bitwise: one
    particle, a chunk just past a block's threads, tiles of several chunks,
    and particles that leave their tile's windows within the call."""
    import torch
    st = _state(n, npart, seed=3 * n + npart)
    times = [0.0, 0.05, 0.1, 0.15]
    out = []
    for tiled in (False, True):
        ctx = pm.PMContext(pm.make_params(n, npart, float(n), hbar_over_m=0.01), device=gpu)
        pos, vel = to_device(st, gpu)
        vel = torch.randn(vel.shape, generator=torch.Generator().manual_seed(n)).to(gpu)
        vel *= move / 0.05
        if tiled:
            order = torch.arange(npart, dtype=torch.int32, device=gpu)
            ctx.sort(pos, vel, order)
        ctx.step(pos, vel, times)
        torch.cuda.synchronize()
        out.append(_rows(pos, vel))
    assert np.array_equal(out[0], out[1])
