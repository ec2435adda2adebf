"""Lattices whose bottom row is long: the heat flux of a state is sampled by one
block of a step, so wide lattices of few rows keep the two launches, whose
thermal tiles share that work; every way to sample gives the same numbers."""
import pytest

from paper_1501_03857_amd import lbboil as L
from test_gpu_autotune_forms import _launches
from test_gpu_one_launch import _domain, _same_state
from test_zz_no_alloc import _case as _noalloc_equals_step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,precision,mode,launches", [
    (1568, 78, L.FP64, L.ISOTHERMAL, 1), (1569, 78, L.FP64, L.ISOTHERMAL, 2), (8000, 15, L.FP32, L.ISOTHERMAL, 2),
    (5376, 8, L.FP64, L.COUPLED, 1), (5377, 8, L.FP64, L.COUPLED, 2), (13700, 4, L.FP32, L.COUPLED, 2),
    (13700, 31, L.FP32, L.COUPLED, 2), (13700, 38, L.FP64, L.COUPLED, 1), (13700, 54, L.FP32, L.COUPLED, 1)])
def test_steps_of_wide_lattices(nx, ny, precision, mode, launches):
    """Chunks of 56 columns: up to 28 for the isothermal launch, up to 96 for
    tiles of lattices under 32 rows.  The launch that ends the sequence is one
    more, two on bottom rows of more than 48 chunks in one-launch steps."""
    print("[gpu-case] wide lattice", nx, ny, precision, mode, flush=True)
    args = _domain(nx, ny, precision, thermal_mode=mode)
    d = L.Domain(*args)
    assert _launches(d) == 4 * launches + (2 if launches == 1 and nx > 48 * 56 else 1)
    one, two = L.Domain(*args), L.Domain(*args).set_tiles(0, 0)
    for n in (1, 0, 34, 1):
        one.step(n)
        two.step(n)
        _same_state(one, two)


def test_batch_of_unequal_rows_samples_each():
    """One row of more than 48 chunks among short ones: the batch's launch over
    the chunks covers every member."""
    print("[gpu-case] batch with one long row", flush=True)
    args = [_domain(nx, ny, L.FP32) for nx, ny in ((2800, 12), (56, 9), (300, 40))]
    b = L.Batch([a[0] for a in args], [a[1] for a in args], [a[2] for a in args])
    for n in (1, 33):
        b.step(n)
    for i, a in enumerate(args):
        _same_state(b.domain(i), L.Domain(*a).step(34))


@pytest.mark.parametrize("nx", [896, 897])
def test_noalloc_samples_long_rows(nx):
    """Bottom rows of up to 16 chunks are sampled by the last launch itself,
    longer ones by a launch before it."""
    import torch

    print("[gpu-case] noalloc, long bottom row", nx, flush=True)
    for n in (1, 6):
        _noalloc_equals_step(torch, L.FP32, nx, 24, n, seed=23)
