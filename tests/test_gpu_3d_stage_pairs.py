"""Pairs of RK4 stages in one launch (large three-dimensional lattices) against
a launch a stage (small ones): a lattice that repeats a small one along its
periodic axes repeats its solution.  Both do the same sums in another order, in
FP64, and round the same stored values, so in FP64 they differ by rounding (a
few 1e-16 a step, bound 1e-13 after 6 steps) and in FP32 by single flips of the
last place of a stored value (6e-8 a step, bound 1e-6).  The sizes give ragged
last tiles along x, y and z, runs of planes of several lengths, a tile that the
lattice fits, walls and periodic y, and frozen flow."""
import numpy as np
import pytest

from paper_1501_03857_amd import lbboil as L
from test_gpu_one_launch import _domain

pytestmark = pytest.mark.gpu


def _make(p, nz, Tb, rho, T):
    d = L.Domain3(p, nz, Tb, rho)
    d.set_fields(rho, None, T)
    return d


@pytest.mark.parametrize("precision,bound", [(L.FP64, 1e-13), (L.FP32, 1e-6)])
@pytest.mark.parametrize("nx,ny,nz,rx,rz,kw", [
    (24, 100, 15, 5, 4, {}), (59, 89, 20, 2, 3, {}), (30, 50, 30, 4, 4, dict(periodic_y=1)), (40, 20, 60, 3, 4, {}),
    (58, 10, 64, 2, 8, {}), (59, 151, 30, 1, 2, {}), (24, 100, 15, 5, 4, dict(thermal_mode=L.THERMAL_ONLY)),
])
def test_stage_pairs_repeat_a_small_lattice(nx, ny, nz, rx, rz, kw, precision, bound):
    print("[gpu-case] 3-D stage pairs", nx, ny, nz, rx, rz, kw, precision, flush=True)
    p, Tb, rho2 = _domain(nx, ny, precision, **kw)
    rng = np.random.default_rng(5)
    rho = np.broadcast_to(np.asarray(rho2).reshape(1, ny, nx), (nz, ny, nx)) * (1 + 0.01 * rng.random((nz, ny, nx)))
    Tb = np.broadcast_to(np.asarray(Tb).reshape(1, nx), (nz, nx)) * (1 + 0.01 * rng.random((nz, nx)))
    T = Tb.min() * (1 + 0.02 * rng.random((nz, ny, nx)))
    small = _make(p, nz, Tb, rho, T).step(6)
    pb = _domain(nx * rx, ny, precision, **kw)[0]
    pb.g = p.g
    big = _make(pb, nz * rz, np.tile(Tb, (rz, rx)), np.tile(rho, (rz, 1, rx)), np.tile(T, (rz, 1, rx))).step(6)
    a, b = small.fields(f=False), big.fields(f=False)
    for k in ("T", "rho"):
        want = np.tile(a[k], (rz, 1, rx))
        assert np.isfinite(b[k]).all()
        assert np.abs(b[k] - want).max() <= bound * np.abs(want).max(), k
    if not kw.get("periodic_y"):
        ha, hb = small.heat_flux(), big.heat_flux()
        assert abs(ha["q_mean"] - hb["q_mean"]) <= 100 * bound * np.abs(ha["q_local"]).max()


@pytest.mark.parametrize("nx,ny,nz,kw", [
    (5, 4, 3, {}), (19, 14, 11, dict(periodic_y=1)), (64, 64, 64, {}), (64, 64, 65, {}),
    (19, 14, 11, dict(thermal_mode=L.ISOTHERMAL)),
])
def test_reductions_do_not_depend_on_how_steps_are_split(nx, ny, nz, kw):
    """rho_ave and the heat-flux samples come from the LB launch's own blocks up
    to 1024 partials (64^3 has 1024, 64 x 64 x 65 more) and from a reduction
    launch at the end of a sequence: the same sums in the same order."""
    print("[gpu-case] 3-D split steps", nx, ny, nz, kw, flush=True)
    p, Tb, rho = _domain(nx, ny, L.FP64, **kw)
    rho = np.broadcast_to(np.asarray(rho).reshape(1, ny, nx), (nz, ny, nx)).copy()
    Tb = np.broadcast_to(np.asarray(Tb).reshape(1, nx), (nz, nx)).copy()
    a, b = L.Domain3(p, nz, Tb, rho), L.Domain3(p, nz, Tb, rho)
    a.step(37)
    q = []
    for n in (1, 1, 32, 0, 3):
        b.step(n)
        q.append(b.heat_flux()["q_now"])
    fa, fb = a.fields(), b.fields()
    for k in ("f", "T", "rho", "ux", "uy", "uz"):
        assert np.array_equal(fa[k], fb[k]), k
    ha, hb = a.heat_flux(), b.heat_flux()
    assert ha["n_samples"] == hb["n_samples"] == 37 and a.t == b.t == 37
    assert ha["q_now"] == hb["q_now"] and ha["q_mean"] == hb["q_mean"]
