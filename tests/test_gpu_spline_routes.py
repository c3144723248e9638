"""The kernels that a spline call can take, by order, size and support: the
same results on each, and none that costs a multiple of another."""

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


def _lattice(n):
    """One particle per cell, in the mesh's order, moved by 0.3 cells (rms)."""
    rng = np.random.default_rng(n)
    i = np.stack(np.meshgrid(*[np.arange(n)] * 3, indexing="ij"), -1).reshape(-1, 3)
    return quantize_state((i + 0.3 * rng.standard_normal(i.shape)) % n, np.zeros(i.shape), n, {})


def _us(fn, reps=5):
    """Shortest GPU time of one call, in us."""
    import torch
    fn()
    best = float("inf")
    for _ in range(reps):
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        a.record()
        fn()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) * 1e3)
    return best


def _force_bound(x, q, n, h):
    """The force in FP64, and the bound of sums of fewer than 1500 terms in
    any order with a few roundings in each."""
    i = np.floor(x).astype(np.int64)
    reach = np.arange(-int(h), int(h) + 2)
    o = np.stack(np.meshgrid(reach, reach, reach, indexing="ij"), -1).reshape(-1, 3)
    d = o[None] - (x - i)[:, None]
    at = (i[:, None] + o[None]) % n
    r = np.sqrt((d * d).sum(-1))
    s = r / h
    slope = np.where(s <= 0.5, -12 * s + 18 * s ** 2, -6 * np.clip(1 - s, 0, None) ** 2)
    term = (q[(at[..., 0] * n + at[..., 1]) * n + at[..., 2]] * 8 / (np.pi * h ** 4) * slope
            / np.maximum(r, 1e-30))[..., None] * d
    return term.sum(1), 1500 * 2.0 ** -24 * np.abs(term).sum(1) + 1e-12


@pytest.mark.parametrize("h", [2.0, 3.01, 5.0])
@pytest.mark.parametrize("npart", [300, (1 << 16) - 1, (1 << 16) + 1])
def test_force_on_every_route(pm, gpu, npart, h):
    """Below and above the counts at which a force changes its kernel, in the
    caller's order and sorted, against sums in FP64 (of 700 particles)."""
    import torch
    n = 32
    st = _random(n, npart, npart)
    q = np.random.default_rng(1).standard_normal(n ** 3).astype(np.float32)
    pick = np.random.default_rng(2).permutation(npart)[:700]
    ref, bound = _force_bound(st.pos[pick], q, n, h)
    for order in (False, True):
        ctx = pm.PMContext(pm.make_params(n, npart, float(n), hbar_over_m=1.0), device=gpu)
        pos, vel = to_device(st, gpu)
        ids = torch.arange(npart, dtype=torch.int32, device=gpu)
        if order:
            ctx.sort(pos, vel, ids)
        acc = torch.empty((3, npart), dtype=torch.float32, device=gpu)
        ctx.spline_qforce(pos, torch.from_numpy(q).to(gpu), acc, h)
        back = torch.empty_like(acc)
        back[:, ids.long()] = acc
        g = back.cpu().numpy().T[pick].astype(np.float64)
        assert np.all(np.abs(g - ref) <= bound)


def test_unsorted_force_loads_its_own_support(pm, gpu):
    """Many particles in random order: the cost follows the support, not the
    half-cell class above it (114 of 180 nodes at h = 3.01 and 3.5)."""
    import torch
    n, npart = 128, 1 << 20
    pos, _ = to_device(_random(n, npart, 3), gpu)
    ctx = pm.PMContext(pm.make_params(n, npart, float(n), hbar_over_m=1.0), device=gpu)
    q, acc = torch.randn(n ** 3, device=gpu), torch.empty((3, npart), device=gpu)
    narrow, wide = (_us(lambda: ctx.spline_qforce(pos, q, acc, h)) for h in (3.01, 3.5))
    assert narrow <= 0.85 * wide


@pytest.mark.parametrize("h", [2.0, 3.5, 5.0])
@pytest.mark.parametrize("npart", [8192 * 4 - 1, 8192 * 4, 8192 * 32 - 1, 8192 * 32])
def test_sparse_sorted_context(pm, gpu, npart, h):
    """8192 tiles (256^3) on both sides of the counts from which their windows
    are used: the density bitwise the unsorted one, the force the same sums
    (bound: each sum's 300 terms rounded in another order), the step's route
    read from its kernels."""
    import torch
    n = 256
    st = _random(n, npart, npart)
    q = torch.randn(n ** 3, generator=torch.Generator(device=gpu).manual_seed(1), device=gpu)
    out = []
    for order in (False, True):
        ctx = pm.PMContext(pm.make_params(n, npart, float(n), hbar_over_m=1e-4), device=gpu)
        pos, vel = to_device(st, gpu)
        ids = torch.arange(npart, dtype=torch.int32, device=gpu)
        if order:
            ctx.sort(pos, vel, ids)
        delta, acc = torch.empty(n ** 3, device=gpu), torch.empty((3, npart), device=gpu)
        ctx.spline_density(pos, delta, h)
        ctx.spline_qforce(pos, q, acc, h)
        ctx.timing(True)
        ctx.spline_step(pos, vel, [0.0, 0.01], h)
        kernels = ctx.timing_read()
        back, v = torch.empty_like(acc), torch.empty_like(vel)
        back[:, ids.long()], v[:, ids.long()] = acc, vel
        out.append((delta, back.double(), v.double(), "force" in kernels))
    assert torch.equal(out[0][0], out[1][0])
    scale = float(out[0][1].abs().max())
    assert float((out[0][1] - out[1][1]).abs().max()) <= 300 * 2.0 ** -24 * 8 * scale
    kick = float((out[0][2] - torch.from_numpy(st.vel32.astype(np.float64)).to(gpu)).abs().max())
    assert float((out[0][2] - out[1][2]).abs().max()) <= 2.0 ** -16 * kick + 2.0 ** -22
    assert out[0][3] and out[1][3] == (npart < 8192 * (64 if h < 2.5 else 32))


@pytest.mark.parametrize("h", [2.0, 3.01, 5.0, 5.3])
@pytest.mark.parametrize("npart,order", [(300, "none"), (70001, "none"), (300, "sorted"),
                                         (70001, "sorted"), (70001, "foreign")])
def test_force_ignores_what_lies_beyond_the_support(pm, gpu, npart, order, h):
    """Values of Q that are not finite, outside a particle's support or on the
    node it sits on: its force is the one with zeros there, in FP64."""
    import torch
    n = 32
    rng = np.random.default_rng(npart)
    x = rng.random((npart, 3)) * n
    x[: npart // 3] = np.floor(x[: npart // 3])     # on a node
    st = quantize_state(x, np.zeros((npart, 3)), n, {})
    bad = rng.random(n ** 3) < (0.005 if h < 4.0 else 0.001)
    q = rng.standard_normal(n ** 3).astype(np.float32)
    zero = np.where(bad, 0.0, q).astype(np.float32)
    q[bad] = rng.choice(np.float32([np.inf, -np.inf, np.nan]), bad.sum())
    # particles (of 4000) with no bad node within h, up to rounding, but for
    # the one they sit on
    pick = rng.permutation(npart)[:4000]
    i = np.floor(st.pos[pick]).astype(np.int64)
    reach = np.arange(-int(h), int(h) + 2)
    clean = np.zeros(npart, dtype=bool)
    clean[pick] = True
    for o in np.stack(np.meshgrid(reach, reach, reach, indexing="ij"), -1).reshape(-1, 3):
        r2 = ((o - (st.pos[pick] - i)) ** 2).sum(1)
        at = (i + o) % n
        clean[pick] &= ~((r2 > 0) & (r2 < (h * (1 + 1e-5)) ** 2)
                         & bad[(at[:, 0] * n + at[:, 1]) * n + at[:, 2]])
    assert 0.1 < clean[pick].mean() < 0.9
    ctx = pm.PMContext(pm.make_params(n, npart, float(n), hbar_over_m=1.0), device=gpu)
    pos, vel = to_device(st, gpu)
    ids = torch.arange(npart, dtype=torch.int32, device=gpu)
    if order == "sorted":
        ctx.sort(pos, vel, ids)
    elif order == "foreign":
        other, _ = to_device(_random(n, npart, 8), gpu)
        ctx.sort(other, vel)
    acc = torch.empty((3, npart), dtype=torch.float32, device=gpu)
    ctx.spline_qforce(pos, torch.from_numpy(q).to(gpu), acc, h)
    back = torch.empty_like(acc)
    back[:, ids.long()] = acc
    own = np.flatnonzero(clean)[:1500]
    ref, bound = _force_bound(st.pos[own], zero, n, h)
    assert np.all(np.abs(back.cpu().numpy().T[own] - ref) <= bound)


def test_positions_that_were_not_the_sorted_ones(pm, gpu):
    """A second state, in the mesh's order, on a context that sorted another:
    the density bitwise and the force the same sums (300 terms rounded in
    another order) as unsorted, neither at a multiple of its cost."""
    import torch
    n, npart, h = 128, 128 ** 3, 3.5
    lp = pm.make_params(n, npart, float(n), hbar_over_m=1.0)
    pos, _ = to_device(_lattice(n), gpu)
    q = torch.randn(n ** 3, generator=torch.Generator(device=gpu).manual_seed(2), device=gpu)
    out = []
    for order in (False, True):
        ctx = pm.PMContext(lp, device=gpu)
        if order:
            other, vel = to_device(_random(n, npart, 4), gpu)
            ctx.sort(other, vel)
        delta, acc = torch.empty(n ** 3, device=gpu), torch.empty((3, npart), device=gpu)
        us = [_us(lambda: ctx.spline_density(pos, delta, h), 3),
              _us(lambda: ctx.spline_qforce(pos, q, acc, h))]
        out.append((delta, acc.double(), us))
    assert torch.equal(out[0][0], out[1][0])
    scale = float(out[0][1].abs().max())
    assert float((out[0][1] - out[1][1]).abs().max()) <= 300 * 2.0 ** -24 * 8 * scale
    assert out[1][2][0] <= 1.25 * out[0][2][0]
    assert out[1][2][1] <= 3.0 * out[0][2][1]


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("n,npart,h,moved", [(16, 20001, 2.0, 1.0), (32, 40001, 3.5, 0.5),
                                             (64, 120001, 5.0, 3.0), (64, 120001, 3.5, 20.0)])
def test_push_of_dense_tiles_and_strays(pm, gpu, n, npart, h, moved, prec):
    """The fused step where tiles hold several pieces and particles have left
    theirs (by a wave each, near or far; by their lanes where many are far),
    against the separate kernels.  Each force is a sum of up to 600 terms
    rounded in another order, whose magnitudes may exceed their sum's by 8."""
    import torch
    rng = np.random.default_rng(npart)
    x = rng.random((npart, 3)) * n
    x[: npart // 2] = 9.0 + 5.0 * rng.random((npart // 2, 3))       # one dense tile
    first = quantize_state(x, np.zeros((npart, 3)), n, {})
    st = quantize_state((x + moved * rng.standard_normal((npart, 3))) % n,
                        0.05 * rng.standard_normal((npart, 3)), n, {})
    lp = pm.make_params(n, npart, float(n), hbar_over_m=0.05, precision=prec)
    out = []
    for fused in (False, True):
        ctx = pm.PMContext(lp, device=gpu)
        pos, vel = to_device(st, gpu, fp32_positions=prec == 0)
        ids = torch.arange(npart, dtype=torch.int32, device=gpu)
        if fused:
            sorted_pos, sorted_vel = to_device(first, gpu, fp32_positions=prec == 0)
            ctx.sort(sorted_pos, sorted_vel, ids)
            pos, vel = pos[:, ids.long()].contiguous(), vel[:, ids.long()].contiguous()
        ctx.timing(True)
        ctx.spline_step(pos, vel, [0.0, 0.01, 0.02], h)
        assert ("force" in ctx.timing_read()) == (not fused)
        p, v = torch.empty_like(pos), torch.empty_like(vel)
        p[:, ids.long()], v[:, ids.long()] = pos, vel
        cells = (p.long() & 0xffffffff).double() * (n / 2.0 ** 32) if prec else p.double()
        out.append((cells, v.double()))
    kick = float((out[0][1] - torch.from_numpy(st.vel32.astype(np.float64)).to(gpu)).abs().max())
    bound = 600 * 2.0 ** -24 * 8 * kick + 2.0 ** -22
    assert float((out[1][1] - out[0][1]).abs().max()) <= bound
    d = (out[1][0] - out[0][0] + n / 2) % n - n / 2
    assert float(d.abs().max()) <= 0.02 * bound + 2.0 ** -22 * n
