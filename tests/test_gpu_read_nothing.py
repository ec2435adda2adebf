"""A read-back of no field waits for the domain's work and checks its state."""
import ctypes as C

import numpy as np
import pytest

from paper_1501_03857_amd import lbboil as L
from test_gpu_capture_reads import _domain3
from test_gpu_one_launch import _domain
from test_gpu_pending_work import _hot, _invalid

pytestmark = pytest.mark.gpu


def _idle(d):
    return L.lib().hipStreamQuery(C.c_void_p(d.stream)) == 0


@pytest.mark.parametrize("dims", [2, 3])
def test_a_read_of_no_field_waits(dims):
    print("[gpu-case] read of no field", dims, flush=True)
    d = L.Domain(*_domain(160, 60, L.FP64)) if dims == 2 else _domain3(L.FP64)
    d.step(32)
    d.step_async(4096)
    if dims == 2:
        assert L.lib().lbb_read_fields(d.handle, L.FIELD_ALL, None, None, None, None, None) == L.LBB_OK
    else:
        assert L.lib().lbb3_read_fields(d._h, None, None, None, None) == L.LBB_OK
    assert _idle(d)


def test_a_read_of_no_field_finds_an_invalid_state():
    d = L.Domain(_hot(), rho0=np.full((8, 16), 6.0))
    _invalid(d)
    d.step(0)
    assert L.lib().lbb_read_fields(d.handle, 0, None, None, None, None, None) == L.LBB_OK
    with pytest.raises(L.LbbError) as e:
        d.sync()
    assert e.value.code == L.LBB_ENONFINITE
