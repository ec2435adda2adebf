"""Autotuning chooses shapes for steps of two launches and leaves the form of
the step alone: lattices that step in one launch still do afterwards."""
import ctypes as C

import pytest

from paper_1501_03857_amd import lbboil as L
from test_gpu_one_launch import _domain, _same_state

pytestmark = pytest.mark.gpu


def _launches(d, n=4):
    """Kernels that step_async(n) enqueues, the one that ends the sequence among them."""
    hip, stream = L.lib(), C.c_void_p(d.stream)
    graph, count = C.c_void_p(), C.c_size_t(0)
    assert hip.hipStreamBeginCapture(stream, 1) == 0  # thread local
    d.step_async(n)
    assert hip.hipStreamEndCapture(stream, C.byref(graph)) == 0
    assert hip.hipGraphGetNodes(graph, None, C.byref(count)) == 0 and hip.hipGraphDestroy(graph) == 0
    return count.value


@pytest.mark.parametrize("nx,ny,precision,mode", [
    (248, 512, L.FP64, L.ISOTHERMAL), (300, 400, L.FP32, L.ISOTHERMAL), (300, 400, L.FP64, L.ISOTHERMAL),
    (256, 128, L.FP64, L.COUPLED)])
def test_autotune_keeps_the_one_launch_step(nx, ny, precision, mode):
    print("[gpu-case] autotune and the one-launch step", nx, ny, precision, mode, flush=True)
    args = _domain(nx, ny, precision, thermal_mode=mode)
    d, ref = L.Domain(*args), L.Domain(*args)
    assert _launches(d) == 5
    d.autotune(20)
    assert _launches(d) == 5
    d.step(33), ref.step(33)
    _same_state(d, ref)
    d.set_tiles(1, 1)
    assert _launches(d) == 9


def test_isothermal_batch_steps_on_after_autotune():
    print("[gpu-case] autotuned isothermal batch", flush=True)
    args = [_domain(160, 60 + k, L.FP64, thermal_mode=L.ISOTHERMAL) for k in range(30)]
    b = L.Batch([a[0] for a in args], [a[1] for a in args], [a[2] for a in args])
    b.autotune(20)
    b.step(35)
    for i in (0, 17, 29):
        _same_state(b.domain(i), L.Domain(*args[i]).step(35))
