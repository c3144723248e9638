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


def _spline_nodes(x, n, h):
    """(node index, offset vectors, r) of every node within reach, FP64."""
    i = np.floor(x).astype(np.int64)
    f = x - i
    reach = np.arange(-int(h), int(h) + 2)
    o = np.stack(np.meshgrid(reach, reach, reach, indexing="ij"), -1).reshape(-1, 3)
    d = o[None] - f[:, None]
    at = (i[:, None] + o[None]) % n
    return (at[..., 0] * n + at[..., 1]) * n + at[..., 2], d, np.sqrt((d * d).sum(-1))


@pytest.mark.parametrize("h", [2.0, 2.5, 2.7, 3.5, 4.0, 4.4, 5.0, 5.3])
@pytest.mark.parametrize("n,npart", [(16, 37), (32, 700)])
def test_spline_reach_classes(pm, gpu, n, npart, h):
    """Density and force at each class of supports, edges included: tiled (a
    sorted context, most particles having left their tile since) against
    direct (bitwise for the density) and against sums in FP64."""
    import torch
    st = _state(n, npart, seed=npart)
    moved = _state(n, npart, seed=npart + 1)
    lp = pm.make_params(n, npart, float(n), hbar_over_m=1.0)
    rng = np.random.default_rng(n)
    q = rng.standard_normal(n ** 3).astype(np.float32)
    dens, force = [], []
    for tiled in (False, True):
        ctx = pm.PMContext(lp, device=gpu)
        pos, vel = to_device(moved, gpu)
        if tiled:   # a tile map of the same count; a third of the particles stay in it
            first, _ = to_device(st, gpu)
            first[:, ::3] = pos[:, ::3]
            ids = torch.arange(npart, dtype=torch.int32, device=gpu)
            ctx.sort(first, vel, ids)
            pos = pos[:, ids.long()].contiguous()
        delta = torch.empty(n ** 3, dtype=torch.float32, device=gpu)
        acc = torch.empty((3, npart), dtype=torch.float32, device=gpu)
        ctx.spline_density(pos, delta, h)
        mass = ctx.workspace[: 8 * n ** 3].view(torch.int64).clone()
        ctx.spline_qforce(pos, torch.from_numpy(q).to(gpu), acc, h)
        torch.cuda.synchronize()
        if tiled:
            back = torch.empty_like(acc)
            back[:, ids.long()] = acc
            acc = back
        dens.append(mass.cpu().numpy())
        force.append(acc.cpu().numpy().T.astype(np.float64))
    assert np.array_equal(dens[0], dens[1])
    at, d, r = _spline_nodes(moved.pos, n, h)
    s = r / h
    c = 8 / (np.pi * h ** 3)
    w = np.where(s <= 0.5, 1 - 6 * s ** 2 + 6 * s ** 3, 2 * np.clip(1 - s, 0, None) ** 3)
    ref = np.bincount(at.ravel(), c * w.ravel(), minlength=n ** 3) * 2.0 ** 40
    hits = np.bincount(at.ravel(), (s < 1).ravel(), minlength=n ** 3)
    # a kernel value takes a few roundings of q <= 1, times a slope below 2:
    # 2^-20 of its maximum c, plus the rounding to integer units
    assert np.all(np.abs(dens[0] - ref) <= hits * (2.0 ** -20 * c * 2.0 ** 40 + 1.0))
    slope = np.where(s <= 0.5, -12 * s + 18 * s ** 2, -6 * np.clip(1 - s, 0, None) ** 2)
    term = (q[at] * c / h * slope / np.maximum(r, 1e-30))[..., None] * d
    # sums of fewer than 1500 terms in any order, a few roundings in each
    bound = 1500 * 2.0 ** -24 * np.abs(term).sum(1) + 1e-12
    for g in force:
        assert np.all(np.abs(g - term.sum(1)) <= bound)


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("n,npart,h", [(16, 1, 2.0), (16, 2500, 3.5), (32, 6000, 4.6)])
def test_spline_push_equals_separate_passes(pm, gpu, n, npart, h, prec):
    """One pass for both forces, kicks and drift (sorted context) against the
    separate kernels (unsorted): the same sums in the same order, so they
    differ by the contraction of a few roundings of partial sums at most."""
    import torch
    st = _state(n, npart, seed=npart, clumps=False)
    lp = pm.make_params(n, npart, float(n), hbar_over_m=0.5, precision=prec)
    out = []
    for fused in (False, True):
        ctx = pm.PMContext(lp, device=gpu)
        pos, vel = to_device(st, gpu, fp32_positions=prec == 0)
        ids = torch.arange(npart, dtype=torch.int32, device=gpu)
        if fused:
            ctx.sort(pos, vel, ids)
        ctx.spline_step(pos, vel, [0.0, 0.01, 0.03], h)
        torch.cuda.synchronize()
        p, v = torch.empty_like(pos), torch.empty_like(vel)
        p[:, ids.long()], v[:, ids.long()] = pos, vel
        x = p.double() * (n / 2.0 ** 32 if prec else 1.0)
        out.append((x.cpu().numpy(), v.cpu().numpy().astype(np.float64)))
    kick = max(np.abs(out[0][1] - st.vel32.astype(np.float64)).max(), 1e-6)
    assert np.abs(out[1][1] - out[0][1]).max() <= 2.0 ** -16 * kick + 2.0 ** -22
    # a position word is one rounding of the drift on top
    d = (out[1][0] - out[0][0] + n / 2) % n - n / 2
    assert np.abs(d).max() <= 0.03 * (2.0 ** -16 * kick + 2.0 ** -22) + 2.0 ** -22 * n


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("n,npart,clumps", [(32, 1 << 17, False), (32, (1 << 17) + 1, True),
                                            (64, 64 ** 3, True)])
def test_binned_deposit_equals_direct(pm, gpu, n, npart, clumps, prec):
    """From 2^17 particles on an unsorted deposit is binned: against the FP64
    sum, and (fixed point) bitwise against halves below the limit deposited
    directly; the second state of the density difference likewise."""
    import torch
    st = _state(n, npart, seed=npart, clumps=clumps)
    ctx = pm.PMContext(pm.make_params(n, npart, float(n), precision=prec), device=gpu)
    pos, vel = to_device(st, gpu, fp32_positions=prec == 0)
    ctx.deposit(pos)
    torch.cuda.synchronize()
    op = oracle.Params(n=n, box=float(n), S=1.0, hbar_m=0.0)
    if prec == 0:
        acc = ctx.workspace[: 4 * n ** 3].view(torch.float32).cpu().numpy().astype(np.float64)
        ref = oracle.deposit(pos.cpu().numpy().T.astype(np.float64), op).ravel() * npart / n ** 3
        # as for the tiled deposit, and one half-ulp for each of the chunks of
        # a tile past the first
        assert np.all(np.abs(acc - ref) <= (11 + npart // 8192) * 2.0 ** -24 * ref + 1e-30)
    else:
        mass = ctx.workspace[: 8 * n ** 3].view(torch.int64).cpu().numpy().copy()
        total = np.zeros(n ** 3, dtype=np.int64)
        for part in np.array_split(np.arange(npart), 3):
            sub = pm.PMContext(pm.make_params(n, len(part), float(n)), device=gpu)
            sub.deposit(pos[:, part[0]: part[-1] + 1].contiguous())
            torch.cuda.synchronize()
            total += sub.workspace[: 8 * n ** 3].view(torch.int64).cpu().numpy()
        assert np.array_equal(mass, total)
    other, _ = to_device(_state(n, npart, seed=npart + 1, clumps=False), gpu,
                         fp32_positions=prec == 0)
    plain = ctx.density_rms_diff(pos, other)
    ctx.sort(pos, vel)
    again = ctx.density_rms_diff(pos, other)
    assert again[1] == plain[1]
    assert abs(again[0] - plain[0]) <= (0.0 if prec else 1e-3) * plain[0] + 1e-12 * plain[0]


@pytest.mark.parametrize("prec", [0, 1])
def test_unsorted_step_with_binned_deposit(pm, gpu, prec):
    """A large unsorted call bins each step's deposit instead of adding from
    the push: against the same state sorted, which never does."""
    import torch
    n, npart = 32, (1 << 17) + 77
    st = _state(n, npart, seed=5, clumps=False)
    out = []
    for tiled in (False, True):
        ctx = pm.PMContext(pm.make_params(n, npart, float(n), hbar_over_m=0.01, precision=prec),
                           device=gpu)
        pos, vel = to_device(st, gpu, fp32_positions=prec == 0)
        ids = torch.arange(npart, dtype=torch.int32, device=gpu)
        if tiled:
            ctx.sort(pos, vel, ids)
        ctx.step(pos, vel, [0.0, 0.05, 0.1, 0.15])
        torch.cuda.synchronize()
        p, v = torch.empty_like(pos), torch.empty_like(vel)
        p[:, ids.long()], v[:, ids.long()] = pos, vel
        out.append((p, v))
    if prec:
        assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
    else:   # float sums of the density differ in order: 2^-20 of it in the force
        kick = float((out[1][1] - torch.from_numpy(st.vel32.copy()).to(gpu)).abs().max())
        assert float((out[0][1] - out[1][1]).abs().max()) <= 1e-3 * kick


@pytest.mark.parametrize("prec", [0, 1])
def test_force_of_combined_potential(pm, gpu, prec):
    """From 2^16 particles on the force reads fg phi + fq Q formed beforehand:
    bitwise the force of parts of the particles that are below the limit."""
    import torch
    n, npart = 32, (1 << 16) + 5
    pos, _ = to_device(_state(n, npart, seed=9), gpu, fp32_positions=prec == 0)
    gen = torch.Generator(device=gpu).manual_seed(1)
    phi, q = (torch.randn(n ** 3, generator=gen, device=gpu) for _ in range(2))

    def force(p):
        lp = pm.make_params(n, p.shape[1], float(n), hbar_over_m=1.0, comoving=True,
                            precision=prec)
        acc = torch.empty(p.shape, dtype=torch.float32, device=gpu)
        ctx = pm.PMContext(lp, device=gpu)
        ctx.force(p, acc, 0.3, phi, q)
        torch.cuda.synchronize()
        return acc

    whole = force(pos)
    parts = torch.cat([force(p.contiguous()) for p in pos.split(30000, dim=1)], dim=1)
    assert torch.equal(whole, parts)


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("n", [16, 32, 64, 128, 256])
def test_last_pass_with_stencil(pm, gpu, n, prec):
    """The Q of the solve's last pass (clumps over empty cells, which the box
    corner crosses) against the stencil alone on the same density, bitwise,
    and phi against the solve alone; both are read through a step's fields."""
    import torch
    npart = n ** 3 // 3 + 1
    st = _state(n, npart, seed=n)
    lp = pm.make_params(n, npart, float(n), hbar_over_m=0.3, precision=prec, comoving=True)
    ctx = pm.PMContext(lp, device=gpu)
    pos, vel = to_device(st, gpu, fp32_positions=prec == 0)
    ctx.sort(pos, vel)
    ctx.step(pos, vel, [0.5, 0.5 + 1e-9])   # leaves phi and Q at the positions
    one, two = torch.empty((3, npart), device=gpu), torch.empty((3, npart), device=gpu)
    ctx.force(pos, one, 0.5)
    phi, q = torch.empty(n ** 3, device=gpu), torch.empty(n ** 3, device=gpu)
    delta = torch.empty(n ** 3, device=gpu)
    if prec:   # (the float deposit is not repeatable to the bit)
        ctx.deposit(pos, delta)
        ctx.poisson(None, phi)
        ctx.qpot(None, q)
        ctx.force(pos, two, 0.5, phi, q)
        torch.cuda.synchronize()
        assert torch.equal(one, two)
    op = oracle.Params(n=n, box=float(n), S=0.45, hbar_m=0.3, comoving=True)
    if n <= 64:
        x = pos.cpu().numpy().T.astype(np.float64) if prec == 0 else None
        if prec:
            from gpu_helpers import positions_cells
            x = positions_cells(pos, n)
        e = ctx.energy(pos, vel, 0.5)
        ref = oracle.energies(x, vel.cpu().numpy().T.astype(np.float64), op, 0.5)
        for key in ("K", "W", "U"):
            assert abs(e[key] - ref[key]) <= 1e-5 * abs(ref[key])


@pytest.mark.parametrize("n", [16, 32, 64])
def test_mesh_outputs_of_the_composable_calls(pm, gpu, n):
    """The meshes a caller gets: written by the kernels (aligned), copied
    (one float off an 8-byte boundary), over the input, and from the spectrum
    that the deposit leaves or from a fresh transform -- the same each time."""
    import torch
    npart = n ** 3 // 2
    ctx = pm.PMContext(pm.make_params(n, npart, float(n), hbar_over_m=0.3), device=gpu)
    pos, _ = to_device(_state(n, npart, seed=2 * n), gpu)
    odd = [torch.empty(n ** 3 + 1, device=gpu)[1:] for _ in range(3)]
    even = [torch.empty(n ** 3, device=gpu) for _ in range(3)]
    for delta, phi, q in (even, odd):
        ctx.deposit(pos, delta)
        ctx.poisson(None, phi)
        ctx.qpot(None, q)
    again = torch.empty(n ** 3, device=gpu)
    ctx.poisson(None, again)            # the spectrum is gone: a fresh transform
    given = torch.empty(n ** 3, device=gpu)
    ctx.poisson(even[0], given)
    over = even[0].clone()
    apart = torch.empty(n ** 3, device=gpu)
    ctx.qpot(over, over)
    ctx.qpot(even[0], apart)
    both = even[0].clone()
    ctx.poisson(both, both)
    torch.cuda.synchronize()
    for a, b in zip(even, odd):
        assert torch.equal(a, b)
    for a in (again, given, both):
        assert torch.equal(a, even[1])
    assert torch.equal(over, apart)
