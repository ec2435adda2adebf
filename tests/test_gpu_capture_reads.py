"""Steps recorded into a caller's graph do not run when they are enqueued: the
domain's scalars stay those of the device until the graph is launched."""
import ctypes as C

import numpy as np
import pytest

from paper_1501_03857_amd import lbboil as L
from test_gpu_one_launch import _domain
from test_gpu_pending_work import _hot, _invalid

pytestmark = pytest.mark.gpu

THREAD_LOCAL = 1  # hipStreamCaptureModeThreadLocal


def _ok(rc):
    assert rc == 0, rc


class _Captured:
    """The work that `record` enqueues on `stream`, as a launchable graph."""

    def __init__(self, stream, record):
        hip, self.stream = L.lib(), C.c_void_p(stream)
        graph, self.exec = C.c_void_p(), C.c_void_p()
        _ok(hip.hipStreamBeginCapture(self.stream, THREAD_LOCAL))
        record()
        _ok(hip.hipStreamEndCapture(self.stream, C.byref(graph)))
        _ok(hip.hipGraphInstantiate(C.byref(self.exec), graph, None, None, C.c_size_t(0)))
        _ok(hip.hipGraphDestroy(graph))

    def launch(self):
        _ok(L.lib().hipGraphLaunch(self.exec, self.stream))

    def close(self):
        _ok(L.lib().hipGraphExecDestroy(self.exec))


def _domain3(precision):
    p, Tb, rho = _domain(19, 14, precision)
    T3 = np.broadcast_to(np.asarray(Tb).reshape(1, 19), (11, 19)).copy()
    return L.Domain3(p, 11, T3, np.broadcast_to(np.asarray(rho).reshape(1, 14, 19), (11, 14, 19)).copy())


@pytest.mark.parametrize("kind", ["tiles", "two launches", "isothermal", "3-D"])
def test_scalars_after_recording_steps(kind):
    print("[gpu-case] steps recorded into a caller's graph", kind, flush=True)

    def make():
        if kind == "3-D":
            return _domain3(L.FP64)
        d = L.Domain(*_domain(70, 37, L.FP64, **(dict(thermal_mode=L.ISOTHERMAL) if kind == "isothermal" else {})))
        return d.set_tiles(0, 0) if kind == "two launches" else d

    d, ref = make(), make()
    for x in (d, ref):
        x.step(5)
        x.reset_average()
    g = _Captured(d.stream, lambda: d.step_async(4))  # an even count: the buffers keep their parity
    assert d.t == 5 and d.heat_flux()["n_samples"] == 0
    for k in range(3):  # replays with the domain's own steps between them
        g.launch()
        ref.step(4)
        a, b = d.heat_flux(), ref.heat_flux()
        assert d.t == ref.t == 9 + 6 * k and a["n_samples"] == b["n_samples"] == 4 + 6 * k
        assert a["q_now"] == b["q_now"] and a["q_mean"] == b["q_mean"]
        d.step(2)
        ref.step(2)
    d.sync()
    g.close()


def test_fields_after_recording_a_read():
    """A read-back into device buffers recorded with the caller's stream: each
    launch reads the state of its time, and what it flags is reported."""
    import torch

    print("[gpu-case] read-back recorded into a caller's graph", flush=True)
    p, Tb, rho = _domain(70, 37, L.FP64)
    d = L.Domain(p, Tb, rho).step(2)
    out = torch.empty((37, 70), dtype=torch.float64, device="cuda")
    other = torch.empty_like(out)
    cs = torch.cuda.Stream()
    d.read_into(T=other.data_ptr(), stream=cs.cuda_stream)
    g = _Captured(cs.cuda_stream, lambda: d.read_into(T=out.data_ptr(), stream=cs.cuda_stream))
    for n in (2, 4, 6):
        d.step(n)
        g.launch()
        cs.synchronize()
        d.read_into(T=other.data_ptr(), stream=cs.cuda_stream)
        cs.synchronize()
        assert torch.equal(out, other) and np.array_equal(out.cpu().numpy(), d.fields()["T"])
        d.sync()
    g.close()
    hot = L.Domain(_hot(), rho0=np.full((8, 16), 6.0))
    _invalid(hot)
    g = _Captured(cs.cuda_stream, lambda: hot.read_into(T=out.data_ptr(), stream=cs.cuda_stream))
    hot.step(0)
    g.launch()
    cs.synchronize()
    with pytest.raises(L.LbbError):
        hot.sync()
    g.close()
