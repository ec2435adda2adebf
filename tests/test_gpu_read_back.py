"""Scalars read from the host copy that the end of a sequence of steps leaves
agree with the device's after every call that changes them: the checkpoint
blob, which is read from the device, is the reference in two dimensions, a
second domain that takes the same steps one at a time in three."""
import numpy as np
import pytest

from paper_1501_03857_amd import lbboil as L
from test_gpu_one_launch import _domain

pytestmark = pytest.mark.gpu


def _reloaded(d, args):
    e = L.Domain(*args)
    e.load(d.save())
    return e


def _agree(d, args):
    e = _reloaded(d, args)
    a, b = d.heat_flux(), e.heat_flux()
    assert a["n_samples"] == b["n_samples"] and d.t == e.t
    assert a["q_now"] == b["q_now"] and np.array_equal(a["q_local"], b["q_local"])
    assert a["q_mean"] == b["q_mean"] or (np.isnan(a["q_mean"]) and np.isnan(b["q_mean"]))


@pytest.mark.parametrize("nx,ny,kw", [(70, 37, {}), (70, 37, dict(periodic_y=1)), (301, 77, {}),
                                      (62, 40, dict(thermal_mode=L.ISOTHERMAL))])
def test_scalars_after_every_call_that_changes_them(nx, ny, kw):
    print("[gpu-case] read back", nx, ny, kw, flush=True)
    args = _domain(nx, ny, L.FP64, **kw)
    d = L.Domain(*args)
    _agree(d, args)
    blob = d.save()
    for change in (lambda: d.step(5), d.reset_average, lambda: d.step(33), lambda: d.step(0),
                   lambda: d.set_heater(np.asarray(args[1]) * 1.001), lambda: d.time_kernels(3),
                   lambda: d.load(blob), lambda: d.step(2)):
        change()
        _agree(d, args)
    if not kw:
        d.adjoint(4, 2)
        _agree(d, args)
    if kw.get("periodic_y"):
        assert not np.any(d.heat_flux()["q_local"])


def test_batch_scalars():
    args = [_domain(n, 40, L.FP64) for n in (70, 60)]
    b = L.Batch([a[0] for a in args], [a[1] for a in args], [a[2] for a in args])
    one = [L.Domain(*a) for a in args]
    for n in (3, 32, 1):
        b.step(n)
        for d in one:
            d.step(n)
        h = b.heat_flux()
        for i, d in enumerate(one):
            assert h["q_now"][i] == d.heat_flux()["q_now"] and h["q_mean"][i] == d.heat_flux()["q_mean"]
    b.domain(0).reset_average()
    b.step(2)
    one[0].reset_average()
    for d in one:
        d.step(2)
    h = b.heat_flux()
    assert [h["q_mean"][i] for i in (0, 1)] == [d.heat_flux()["q_mean"] for d in one]


@pytest.mark.parametrize("precision", [L.FP64, L.FP32])
def test_three_dimensional_scalars_and_fields(precision):
    nx, ny, nz = 19, 14, 11
    p, Tb, rho = _domain(nx, ny, precision)
    rho0 = np.broadcast_to(np.asarray(rho).reshape(1, ny, nx), (nz, ny, nx)).copy()
    T3 = np.broadcast_to(np.asarray(Tb).reshape(1, nx), (nz, nx)).copy()
    a, b = L.Domain3(p, nz, T3, rho0), L.Domain3(p, nz, T3, rho0)
    a.step(7)
    for _ in range(7):
        b.step(1)
    ha, hb = a.heat_flux(), b.heat_flux()
    assert a.t == b.t == 7 and ha["n_samples"] == hb["n_samples"] == 7
    assert ha["q_now"] == hb["q_now"] and ha["q_mean"] == hb["q_mean"]
    # the sample is the mean of the local flux: sums of nx nz terms in another order
    q = np.asarray(ha["q_local"])
    assert abs(q.mean() - ha["q_now"]) <= 4 * q.size * 2.3e-16 * np.abs(q).max()
    a.reset_average()
    assert a.heat_flux()["n_samples"] == 0 and np.isnan(a.heat_flux()["q_mean"])
    with_f, without = a.fields(), a.fields(f=False)
    for k in without:
        if without[k] is not None and k != "f":
            assert np.array_equal(with_f[k], without[k]), k
