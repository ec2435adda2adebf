"""The adjoint's launch forms give one gradient: a lattice alone takes small
temperature tiles and the LB adjoint in one launch, the same lattice among
enough others larger tiles and two launches.  The per-node arithmetic is the
same and every sum over a lattice has an order that neither depends on, so the
results must be bitwise equal.  Sizes: below one tile, ragged last tiles and
columns, lattices smaller than the halo."""
import numpy as np
import pytest

from paper_1501_03857_amd import lbboil as L
from test_gpu_one_launch import _domain

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [L.FP64, L.FP32])
@pytest.mark.parametrize("nx,ny,members", [(3, 5, 1100), (49, 6, 600), (61, 35, 300), (121, 35, 100), (300, 77, 40)])
def test_a_lattice_among_many_has_the_gradient_it_has_alone(nx, ny, members, precision):
    print("[gpu-case] adjoint forms", nx, ny, members, precision, flush=True)
    args = _domain(nx, ny, precision)
    b = L.Batch([args[0]] * members, [args[1]] * members, [args[2]] * members)
    b.step(3)
    J, g, gw = b.adjoint(4, K=2)
    b.close()
    d = L.Domain(*args).step(3)
    Js, gs, gws = d.adjoint(4, K=2)
    assert np.isfinite(gs).all() and np.any(gs != 0.0)
    for i in (0, members // 2, members - 1):
        assert J[i] == Js and np.array_equal(g[i], gs) and gw[i] == gws, i
    # one segment stores every state instead of recomputing: same states
    J1, g1, gw1 = d.adjoint(4, K=4)
    assert J1 == Js and np.array_equal(g1, gs) and gw1 == gws
