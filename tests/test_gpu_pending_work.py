"""What the calls that answer from the host copy of a domain's scalars have to
wait for, and when that copy must not be used."""
import numpy as np
import pytest

from paper_1501_03857_amd import lbboil as L
from test_gpu_one_launch import _domain

pytestmark = pytest.mark.gpu


def _say(*a):
    print("[gpu-case]", *a, flush=True)


# Above T_c a dense state has a negative pseudopotential radicand.
A_HOT = 3.0 / 49.0
RHO_INVALID = 8.5


def _hot(nx=16, ny=8):
    return L.Params(nx=nx, ny=ny, a=A_HOT, Ts_over_Tc=1.1, periodic_y=1, thermal_mode=L.ISOTHERMAL, rho_L=6.5,
                    rho_V=0.4, liquid_rows=4)


def _invalid(d):
    tc, _ = L.eos_constants(A_HOT, 2.0 / 21.0, 1.0, 0.344)
    shape = (d.p.ny, d.p.nx)
    d.set_fields(np.full(shape, RHO_INVALID), T=np.full(shape, 1.1 * tc))


def _pair(n=2):
    args = [_domain(160, 60, L.FP64) for _ in range(n)]
    return L.Batch([a[0] for a in args], [a[1] for a in args], [a[2] for a in args]), [L.Domain(*a) for a in args]


@pytest.mark.parametrize("call", ["sync", "heat_flux"])
def test_batch_call_waits_for_a_member_stepped_alone(call):
    """A member's own pending steps (an even count: the batch may step on) are
    over when a waiting call of the batch returns, and its scalars are theirs."""
    _say("batch", call, "after a member's own steps")
    b, one = _pair()
    b.step(3)
    b.domain(0).step_async(4096)
    h = b.heat_flux() if call == "heat_flux" else b.sync()
    one[0].step(4099)
    one[1].step(3)
    h = h or b.heat_flux()
    for i, d in enumerate(one):
        assert h["q_now"][i] == d.heat_flux()["q_now"] and h["q_mean"][i] == d.heat_flux()["q_mean"]
        assert h["n_samples"][i] == d.heat_flux()["n_samples"]
    b.step(32)
    for i, d in enumerate(one):
        assert b.domain(i).save() == d.step(32).save()


def test_member_call_waits_for_the_steps_of_its_batch():
    _say("member calls after a batch's steps")
    b, one = _pair()
    b.step(2)
    b.step_async(2048)
    got = [(b.domain(i).t, b.domain(i).heat_flux(local=False)) for i in (0, 1)]
    for d, (t, h) in zip(one, got):
        e = d.step(2050).heat_flux()
        assert t == d.t == 2050 and all(h[k] == e[k] for k in ("q_now", "q_mean", "n_samples"))


def test_batch_sync_reports_a_member_that_fails_alone():
    _say("batch sync, failing member")
    b = L.Batch([_hot(), _hot()], None, [np.full((8, 16), 6.0)] * 2)
    b.step(2)
    _invalid(b.domain(1))
    b.domain(1).step_async(2)
    with pytest.raises(L.LbbError) as e:
        b.sync()
    assert e.value.code == L.LBB_ENONFINITE and "member 1" in str(e.value)


@pytest.mark.parametrize("read", ["host", "device", "one field"])
def test_a_read_that_finds_an_invalid_state_is_reported_by_sync(read):
    """The state after the last step is checked by whatever reads it next: a
    read-back flags it, and the next synchronising call reports it."""
    import torch

    _say("invalid state found by a read", read)
    d = L.Domain(_hot(), rho0=np.full((8, 16), 6.0))
    _invalid(d)
    d.step(0)  # ends a sequence of steps; steps nothing, so nothing is checked
    if read == "host":
        d.fields()
    elif read == "one field":
        d.bottom_temperature()
    else:
        rho = torch.empty((8, 16), dtype=torch.float64, device="cuda")
        d.read_into(rho=rho.data_ptr(), stream=torch.cuda.current_stream().cuda_stream)
    with pytest.raises(L.LbbError) as e:
        d.sync()
    assert e.value.code == L.LBB_ENONFINITE


def test_a_member_read_that_finds_an_invalid_state_is_reported_by_its_batch():
    _say("invalid state found by a member's read")
    b = L.Batch([_hot(), _hot()], None, [np.full((8, 16), 6.0)] * 2)
    _invalid(b.domain(1))
    b.step(0)
    for i in (0, 1):
        b.domain(i).fields()
    for _ in range(2):
        with pytest.raises(L.LbbError) as e:
            b.sync()
        assert e.value.code == L.LBB_ENONFINITE and "member 1" in str(e.value)


@pytest.mark.parametrize("recover", ["set_fields", "load"])
def test_a_new_state_clears_what_a_read_found(recover):
    _say("recovery after a read that found an invalid state", recover)
    d = L.Domain(_hot(), rho0=np.full((8, 16), 6.0))
    blob = d.save()
    _invalid(d)
    d.step(0)
    d.fields()
    if recover == "load":
        d.load(blob)
    else:
        d.set_fields(np.full((8, 16), 6.0))
    d.step(3)
    d.fields()
    d.sync()


def test_batch_reports_a_member_read_into_device_memory():
    import torch

    _say("batch sync after a member's device read")
    b = L.Batch([_hot(), _hot()], None, [np.full((8, 16), 6.0)] * 2)
    _invalid(b.domain(1))
    b.step(0)
    out = torch.empty((2, 8, 16), dtype=torch.float64, device="cuda")
    for i in (0, 1):
        b.domain(i).read_into(rho=out[i].data_ptr(), stream=torch.cuda.current_stream().cuda_stream)
    with pytest.raises(L.LbbError) as e:
        b.sync()
    assert e.value.code == L.LBB_ENONFINITE and "member 1" in str(e.value)
