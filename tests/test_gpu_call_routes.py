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


@pytest.mark.parametrize("n,least,least_step,least_four",
                         [(32, 1 << 17, 1 << 17, 1 << 17), (128, 3 << 16, 1 << 18, 1 << 17),
                          (256, 3 << 17, 1 << 19, 1 << 17)])
def test_binning_by_particles_and_mesh(pm, gpu, n, least, least_step, least_four):
    """An unsorted deposit is binned where the particles pay for the mesh's
    tiles, on its own, within a step and for the four of the kinetic split
    (route read from the kernels); the masses and states are bitwise the
    sorted context's."""
    import torch
    for npart in (least_four - 1, least_four, least - 1, least, least_step - 1, least_step):
        st = _random(n, npart, npart)
        lp = pm.make_params(n, npart, float(n), hbar_over_m=1e-3)
        out = []
        for order in (False, True):
            ctx = pm.PMContext(lp, device=gpu)
            pos, vel = to_device(st, gpu)
            ids = torch.arange(npart, dtype=torch.int32, device=gpu)
            if order:
                ctx.sort(pos, vel, ids)
            binned = []
            ctx.timing(True)
            split = ctx.kinetic_split(pos, vel)
            binned.append("sort_count" in ctx.timing_read())
            ctx.timing(True)
            ctx.deposit(pos)
            binned.append("sort_count" in ctx.timing_read())
            mass = ctx.workspace[: 8 * n ** 3].view(torch.int64).clone()
            ctx.timing(True)
            ctx.step(pos, vel, [0.0, 1e-3])     # two deposits: the opening one and the step's
            binned.append(ctx.timing_read().get("sort_count", (0,))[0])
            p, v = torch.empty_like(pos), torch.empty_like(vel)
            p[:, ids.long()], v[:, ids.long()] = pos, vel
            out.append((mass, p, v, split["K"]))
            assert binned == ([False, False, 0] if order
                              else [npart >= least_four, npart >= least,
                                    (npart >= least) + (npart >= least_step)])
            ctx.close()
        assert all(torch.equal(a, b) for a, b in zip(out[0][:3], out[1][:3]))
        assert abs(out[0][3] - out[1][3]) <= 1e-12 * out[1][3]


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("n,npart", [(16, 7), (64, 3000), (128, 70001), (256, 100003), (512, 70001)])
def test_last_pass_on_a_mostly_empty_mesh(pm, gpu, n, npart, prec):
    """phi and Q of the solve's last pass with the stencil, where most cells
    and whole rows are empty, through a step's fields: in the fixed-point form
    bitwise the force of the separate calls.  In the float form each path has
    its own float deposit (one rounding per add, 2^-20 of the density), which
    Q amplifies where cells are nearly empty; with such cells at the floor
    (1e-2) Q's share of the force is bounded by 2^-20 (1 / 1e-2) of its
    largest, and phi's by 2^-20 sqrt(N^3) of it (the solve's rounding)."""
    import torch
    st = _random(n, npart, n + npart)
    lp = pm.make_params(n, npart, float(n), hbar_over_m=0.3, precision=prec,
                        rho_floor=1e-6 if prec else 1e-2)
    ctx = pm.PMContext(lp, device=gpu)
    pos, vel = to_device(st, gpu, fp32_positions=prec == 0)
    ctx.sort(pos, vel)
    vel.zero_()
    ctx.step(pos, vel, [0.0, 1e-30])      # leaves phi and Q at the same positions
    one, two = torch.empty((3, npart), device=gpu), torch.empty((3, npart), device=gpu)
    ctx.force(pos, one)
    phi, q = torch.empty(n ** 3, device=gpu), torch.empty(n ** 3, device=gpu)
    ctx.deposit(pos)
    ctx.poisson(None, phi)
    ctx.qpot(None, q)
    ctx.force(pos, two, 1.0, phi, q)
    torch.cuda.synchronize()
    assert torch.isfinite(two).all() and float(q.abs().max()) > 0.0
    if prec:
        assert torch.equal(one, two)
    else:
        bound = 2.0 ** -20 * (100.0 * float(q.abs().max()) + n ** 1.5 * float(phi.abs().max()))
        assert float((one - two).abs().max()) <= bound


def test_empty_cells_share_the_floor_s_root(pm, gpu):
    """The last pass on a mesh of empty cells costs their masses' loads, not
    six FP64 roots a cell: 2.1 of its time on a filled mesh at 256^3 (2.8 with
    the roots)."""
    import torch
    n = 256
    us = []
    for npart in (1000, n ** 3):
        ctx = pm.PMContext(pm.make_params(n, npart, float(n), hbar_over_m=1e-6), device=gpu)
        if npart == 1000:
            pos, vel = to_device(_random(n, npart, 1), gpu)
        else:
            i = torch.arange(npart, dtype=torch.int32, device=gpu)
            pos = torch.stack([i // n ** 2, i // n % n, i % n]) * (1 << 24) + (1 << 23)
            pos, vel = pos.contiguous(), torch.zeros((3, npart), device=gpu)
        best = float("inf")
        for _ in range(5):
            ctx.timing(True)
            ctx.step(pos, vel, [0.0, 1e-30])
            calls, ms = ctx.timing_read()["c2r_q"]
            best = min(best, ms / calls)
        us.append(best * 1e3)
        ctx.close()
    assert us[0] <= 2.45 * us[1], us


def test_closing_half_kick_of_few_particles(pm, gpu):
    """Too few unsorted particles for one combined potential: the half-kick
    reads two fields, for about three times the cost of one (4.3 with the
    loads in small groups)."""
    import torch
    n, npart = 256, 1 << 20
    pos, vel = to_device(_random(n, npart, 6), gpu)
    us = []
    for hm in (0.0, 1e-6):
        ctx = pm.PMContext(pm.make_params(n, npart, float(n), hbar_over_m=hm), device=gpu)
        best = float("inf")
        for _ in range(6):
            ctx.timing(True)
            ctx.step(pos, vel, [0.0, 1e-30])
            kernels = ctx.timing_read()
            assert "combine" not in kernels
            best = min(best, kernels["kick"][1])
        us.append(best * 1e3)
        ctx.close()
    assert us[1] <= 3.7 * us[0], us


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("n,npart", [(32, (1 << 17) - 1), (32, 1 << 17), (128, 1 << 21),
                                     (128, (1 << 21) + 77), (256, 3000001)])
def test_density_difference_by_the_order_of_each_state(pm, gpu, n, npart, prec):
    """On a sorted context: with many particles a state is binned where it is
    not in the order of the sort and read from its tiles where it is; below,
    b is binned, or nothing (route from the number of binnings).  The
    difference is the unsorted context's."""
    import torch
    lp = pm.make_params(n, npart, float(n), precision=prec)
    ctx, plain = pm.PMContext(lp, device=gpu), pm.PMContext(lp, device=gpu)
    own, vel = to_device(_random(n, npart, 1), gpu, fp32_positions=prec == 0)
    ctx.sort(own, vel)
    near = own.clone()        # a snapshot a little later
    near += (1 << 20) if prec else 1e-3
    other, _ = to_device(_random(n, npart, 2), gpu, fp32_positions=prec == 0)
    for a, b, foreign in ((own, near, 0), (own, other, 1), (other, own, 1), (other, other, 2)):
        rms, cells = plain.density_rms_diff(a, b)
        ctx.timing(True)
        got, got_cells = ctx.density_rms_diff(a, b)
        kernels = ctx.timing_read()
        want = foreign if npart > 1 << 21 else int(npart >= 1 << 17)
        assert kernels.get("sort_scatter", (0, 0))[0] == want
        assert got_cells == cells
        # (float sums of the density in another order: 2^-20 of it, a node)
        assert abs(got - rms) <= (0.0 if prec else 1e-3) * rms + (1e-12 * rms if prec else 1e-5)


def _one_dense_tile(n, npart, seed, gpu):
    """Fixed-point positions, nine tenths of them within one tile."""
    import torch
    gen = torch.Generator(device=gpu).manual_seed(seed)
    x = torch.rand((3, npart), generator=gen, device=gpu, dtype=torch.float64) * n
    dense = npart // 10 * 9
    x[:, :dense] = 8.5 + 6.0 * x[:, :dense] / n
    x = x[:, torch.randperm(npart, generator=gen, device=gpu)]
    u = (x * (2.0 ** 32 / n)).long()
    return torch.where(u >= 2 ** 31, u - 2 ** 32, u).to(torch.int32).contiguous()


@pytest.mark.parametrize("n,npart", [(16, 5), (16, 32768), (64, 300001), (128, 1 << 20)])
def test_lists_of_a_dense_tile(pm, gpu, n, npart):
    """Chunks and pieces of one dense tile among empty and sparse ones cover
    every particle once: deposit and spline density bitwise the direct ones."""
    import torch
    lp = pm.make_params(n, npart, float(n), hbar_over_m=0.1)
    out = []
    for order in (False, True):
        ctx = pm.PMContext(lp, device=gpu)
        pos, vel = _one_dense_tile(n, npart, 1, gpu), torch.zeros((3, npart), device=gpu)
        if order:
            ctx.sort(pos, vel)
        delta = torch.empty(n ** 3, device=gpu)
        ctx.deposit(pos)
        mass = ctx.workspace[: 8 * n ** 3].view(torch.int64).clone()
        assert int(mass.sum()) == npart << 40
        ctx.spline_density(pos, delta, 2.0)
        out.append((mass, delta))
        ctx.close()
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])


def test_scan_of_a_dense_tile(pm, gpu):
    """The scan of a sort does not follow the densest tile: 15 million
    particles in one tile within four times a uniform state's."""
    import torch
    n, npart = 256, 256 ** 3
    vel = torch.zeros((3, npart), device=gpu)
    us = []
    for dense in (False, True):
        ctx = pm.PMContext(pm.make_params(n, npart, float(n)), device=gpu)
        pos = _one_dense_tile(n, npart, 1, gpu) if dense else \
            torch.randint(-2 ** 31, 2 ** 31, (3, npart), dtype=torch.int32, device=gpu)
        best = float("inf")
        for _ in range(4):
            ctx.timing(True)
            ctx.sort(pos.clone(), vel)
            best = min(best, ctx.timing_read()["sort_scan"][1] * 1e3)
        us.append(best)
        ctx.close()
    assert us[1] <= 4.0 * us[0], us
