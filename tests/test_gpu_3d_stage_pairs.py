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
