"""The one-launch step (tiles, k_step, and marching strips, k_march) against
the two launches per step it stands for: the same expressions on the same operands and exact mass sums, so the
state, the heat-flux history and the checkpoint blob must agree bit for bit,
whatever mix of graph replays and single launches made the steps.  The sizes
reach every block shape (16, 32, 48 and 64 region rows) with ragged last tile
columns and rows, one tile, lattices smaller than the halo, and the largest
lattice whose tiles fit one round; strips from the smallest lattice that takes
them on, with ragged last strips, rows and blocks; walls, periodic y and the
ghost layer."""
import numpy as np
import pytest

from paper_1501_03857_amd import lbboil as L
from paper_1501_03857_amd import workloads as WL
from parity_utils import compare, make_pair

pytestmark = pytest.mark.gpu


def _say(*a):
    print("[gpu-case]", *a, flush=True)


def _domain(nx, ny, precision, **kw):
    w = WL.PLAIN_128x64.resized(nx, ny, heater=(nx // 5, nx - nx // 5), seed=11)
    Tc, _ = L.eos_constants(w.a, w.b, w.R, w.omega)
    rv, rl = L.coexistence(w.a, w.b, w.R, w.omega, w.Ts_over_Tc * Tc)
    p = L.Params(nx=nx, ny=ny, precision=precision, liquid_rows=w.liquid_rows, g=WL.scaled_gravity(ny, w.a),
                 Gw_bottom=0.05, Gw_top=-0.03, rho_L=rl, rho_V=rv, **kw)
    return p, w.heater_T(Tc), w.density(rl, rv)


def _same_state(a, b):
    assert a.save() == b.save()
    fa, fb = a.fields(), b.fields()
    for k in ("f", "T", "rho", "ux", "uy"):
        assert np.array_equal(fa[k], fb[k]), k
    ha, hb = a.heat_flux(), b.heat_flux()
    assert ha["q_mean"] == hb["q_mean"] and ha["q_now"] == hb["q_now"] and ha["n_samples"] == hb["n_samples"]
    assert a.t == b.t


@pytest.mark.parametrize("precision", [L.FP64, L.FP32])
@pytest.mark.parametrize("nx,ny,kw", [
    (3, 4, {}), (3, 3, dict(periodic_y=1)), (54, 6, {}), (55, 23, {}), (20, 40, dict(periodic_y=1)),
    (70, 37, dict(periodic_y=1)), (100, 37, dict(ghost_layer=1)), (300, 77, {}), (600, 151, {}),
    (601, 150, dict(periodic_y=1)), (511, 257, {}), (800, 380, {}), (1024, 512, {}), (1080, 513, {}),
    (160, 60, dict(thermal_mode=L.ISOTHERMAL)), (62, 5, dict(thermal_mode=L.ISOTHERMAL)),
    (63, 33, dict(thermal_mode=L.ISOTHERMAL, periodic_y=1)), (248, 512, dict(thermal_mode=L.ISOTHERMAL)),
    (249, 512, dict(thermal_mode=L.ISOTHERMAL)), (90, 40, dict(thermal_mode=L.THERMAL_ONLY)),
])
def test_one_launch_equals_two_launches_bitwise(nx, ny, kw, precision):
    _say("one launch vs two", nx, ny, kw, precision)
    args = _domain(nx, ny, precision, **kw)
    one, two = L.Domain(*args), L.Domain(*args)
    two.set_tiles(0, 0)  # a caller's shapes: two launches per step
    for n in (64, 7, 1, 0, 1, 33):
        one.step(n)
        two.step(n)
    _same_state(one, two)


@pytest.mark.parametrize("precision,nx,ny,kw", [
    (L.FP64, 1250, 1000, {}), (L.FP64, 1733, 767, dict(periodic_y=1)), (L.FP64, 8192, 150, dict(ghost_layer=1)),
    (L.FP32, 2050, 1500, {}), (L.FP32, 3001, 1103, dict(periodic_y=1)), (L.FP32, 1201, 2600, dict(ghost_layer=1)),
    (L.FP32, 4096, 2048, {}), (L.FP32, 8193, 400, {}), (L.FP64, 9000, 31, {}),
])
def test_marching_strips_equal_two_launches_bitwise(precision, nx, ny, kw):
    _say("marching strips vs two launches", precision, nx, ny, kw)
    args = _domain(nx, ny, precision, **kw)
    one, two = L.Domain(*args), L.Domain(*args)
    two.set_tiles(0, 0)
    for n in (33, 2, 0, 1):
        one.step(n)
        two.step(n)
    _same_state(one, two)


@pytest.mark.parametrize("precision,sizes", [
    (L.FP32, [(512, 256), (384, 192), (256, 128), (100, 61), (1024, 33)] * 9),
    (L.FP64, [(512, 256), (384, 193), (256, 128)] * 6),
    (L.FP32, [(512, 256), (384, 192), (256, 31)] * 12),
])
def test_marching_batch_equals_members_alone(precision, sizes):
    """Batches large enough for marching strips (the last has a lattice of too
    few rows for them): each member as alone, where it takes tiles."""
    _say("marching batch", precision, len(sizes))
    args = [_domain(nx, ny, precision) for nx, ny in dict.fromkeys(sizes)]
    mem = [args[list(dict.fromkeys(sizes)).index(x)] for x in sizes]
    b = L.Batch([m[0] for m in mem], [m[1] for m in mem], [m[2] for m in mem]).step(37)
    for i, m in enumerate(args):
        d = L.Domain(*m).step(37)
        for k in (i, len(mem) - len(args) + i):
            _same_state(b.domain(k), d)


@pytest.mark.parametrize("precision", [L.FP64, L.FP32])
@pytest.mark.parametrize("mode", [L.COUPLED, L.ISOTHERMAL])
def test_one_launch_batch_equals_members_alone(precision, mode):
    """A batch whose lattices fit one round together steps in tiles of its own
    height; a change of heater and wall strength between the calls."""
    _say("one-launch batch", precision, mode)
    mem = [_domain(nx, ny, precision, thermal_mode=mode) for nx, ny in ((128, 64), (100, 37), (256, 60), (3, 4), (62, 9))]
    b = L.Batch([m[0] for m in mem], [m[1] for m in mem], [m[2] for m in mem])
    doms = [L.Domain(*m) for m in mem]
    doms[1].set_tiles(1, 2)
    b.step(45)
    b.domain(2).set_wettability(0.11)
    b.domain(0).set_heater(mem[0][1] * 1.01)
    b.step(20)
    for i, d in enumerate(doms):
        d.step(45)
        if i == 2:
            d.set_wettability(0.11)
        if i == 0:
            d.set_heater(mem[0][1] * 1.01)
        d.step(20)
        _same_state(b.domain(i), d)


@pytest.mark.parametrize("precision,tol", [(L.FP64, 1e-12), (L.FP32, 1e-5)])
def test_one_launch_matches_oracle(precision, tol):
    _say("one launch vs oracle", precision)
    w = WL.PLAIN_128x64.resized(130, 61, heater=(30, 90), Gw_bottom=0.05)
    o, d, _ = make_pair(w, precision=precision, Gw_top=-0.03)
    o.step(70)
    d.step(70)
    errs, bad = compare(o, d, tol)
    assert not bad, errs


@pytest.mark.parametrize("precision", [L.FP64, L.FP32])
@pytest.mark.parametrize("K", [0, 5])
def test_adjoint_forward_in_one_launch_equals_two(precision, K):
    """The adjoint's stored states come from the same steps: J and the
    gradients agree bit for bit, and the domain steps on as before."""
    _say("one-launch adjoint", precision, K)
    args = _domain(100, 45, precision)
    one, two = L.Domain(*args).step(9), L.Domain(*args)
    two.set_tiles(0, 0).step(9)
    a, b = one.adjoint(13, K), two.adjoint(13, K)
    assert a[0] == b[0] and np.array_equal(a[1], b[1]) and a[2] == b[2]
    one.step(35)
    two.step(35)
    _same_state(one, two)


@pytest.mark.parametrize("precision", [L.FP64, L.FP32])
def test_noalloc_one_launch_hands_out_density_and_velocity(precision):
    """rho, vx and vy of the last step's old state in the caller's buffers,
    velocity zero on the wall rows.  Bound: one rounding to the storage type
    (2^-24, 2^-53), and a few ulp between the refined reciprocal of the step
    and the division of the read-back."""
    import torch

    _say("noalloc density and velocity", precision)
    nx, ny, n = 130, 37, 6
    p, Tb, rho0 = _domain(nx, ny, precision)
    d = L.Domain(p, Tb, rho0)
    dt = torch.float64 if precision == L.FP64 else torch.float32
    W = torch.tensor([4 / 9] + [1 / 9] * 4 + [1 / 36] * 4, dtype=torch.float64).view(9, 1, 1)
    Tc, _ = L.eos_constants(p.a, p.b, p.R, p.omega)
    T = np.full((ny, nx), p.Ts_over_Tc * Tc)
    T[0] = Tb
    T -= 0.0 if precision == L.FP64 else p.Ts_over_Tc * Tc
    f = [(W * torch.from_numpy(rho0)).to(dt).cuda() for _ in range(2)]
    Ts = [torch.from_numpy(T).to(dt).cuda() for _ in range(2)]
    aux = [torch.full((ny, nx), float("nan"), dtype=dt, device="cuda") for _ in range(3)]
    res = torch.zeros(5, dtype=torch.float64, device="cuda")
    L.step_noalloc(p, [x.data_ptr() for x in f], [x.data_ptr() for x in Ts], *(x.data_ptr() for x in aux), [0, 0], n,
                   res.data_ptr(), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    ref = d.step(n - 1).fields()
    got = [x.double().cpu().numpy() for x in aux]
    eps = 2.0**-52 if precision == L.FP64 else 2.0**-23
    assert np.max(np.abs(got[0] - ref["rho"])) <= 4 * eps * np.max(ref["rho"])
    for g, k in ((got[1], "ux"), (got[2], "uy")):
        assert np.all(g[[0, -1]] == 0.0)
        # the domain's populations at step n - 1 are the same; only the
        # quotient and the storage rounding differ
        assert np.max(np.abs(g[1:-1] - ref[k][1:-1])) <= 8 * eps * np.max(np.abs(ref[k])) + 1e-16, k
