"""lbb_batch_init refuses what lbb_init_domain refuses, by the member's own
error and before anything is allocated (these run without a GPU)."""
import numpy as np
import pytest

from paper_1501_03857_amd import lbboil as L


def _error(params, rho0s=None, T_bottoms=None):
    with pytest.raises(L.LbbError) as e:
        L.Batch(params, T_bottoms, rho0s)
    return e.value.code, str(e.value)


@pytest.mark.parametrize("bad", [dict(nx=2_000_000_000), dict(nx=-5), dict(ny=2), dict(precision=7), dict(G=1.0)])
def test_an_invalid_member_is_named(bad):
    if "precision" in bad:  # shared by all members
        code, text = _error([L.Params(nx=16, ny=8, **bad), L.Params(nx=16, ny=8, **bad)])
        assert code == L.LBB_EINVAL and "member 0" in text
        return
    code, text = _error([L.Params(**{**dict(nx=16, ny=8, liquid_rows=1), **bad}), L.Params(nx=16, ny=8, liquid_rows=1)])
    assert code == L.LBB_EINVAL and "member 0" in text


def test_members_are_checked_in_their_order():
    rho = np.full((8, 16), -1.0)
    code, text = _error([L.Params(nx=16, ny=8, liquid_rows=4), L.Params(nx=2_000_000_000, ny=8)], [rho, None])
    assert code == L.LBB_EINVAL and "member 0" in text and "density" in text


def test_budget_refuses_a_member_first():
    lib = L.lib()
    assert lib.lbb_set_device_budget(1 << 20) == L.LBB_OK
    try:
        code, text = _error([L.Params(nx=512, ny=256)])
        assert code == L.LBB_ENOMEM and "budget" in text and lib.lbb_device_bytes_held() == 0
    finally:
        assert lib.lbb_set_device_budget(0) == L.LBB_OK
