"""Setting a state with and without its CFL maximum (steps of imposed or fixed
dt do without it): the same states, and the same dt once the CFL rule is used
again (needs an MI355X)."""
from __future__ import annotations

import numpy as np
import pytest

import workloads as W
from tests.test_gpu_batch import m2c  # noqa: F401

pytestmark = pytest.mark.gpu


def _problems():
    moving = W.shock_bubble(1, nxyz=(20, 18, 17), radius=0.2, p_shock=1e9, shock_x=0.3)
    return [W.shock_tube_1d(0, nx=37), moving, W.shock_bubble(2, nxyz=(130, 97, 90), radius=0.3),
            W.eos_charge(3, n=(24, 22, 20))]


@pytest.mark.parametrize("k", range(4))
def test_with_and_without_the_maximum(m2c, k):  # noqa: F811
    p = _problems()[k]
    cfg = m2c.config_for(p)
    a = m2c.Sim(cfg, p.prim)
    w0 = a.get_conserved()
    assert a.step(1) == 0
    dt, w1 = a.stats()["dt_last"], a.get_conserved()
    assert dt > 0.0 and np.isfinite(dt)
    a.set_state(p.prim)                       # with it
    assert a.step_dt(1, dt) == 0
    assert np.array_equal(a.get_conserved(), w1)
    for _ in range(2):
        a.set_state(p.prim)                   # without: the last step had its dt imposed
        assert np.array_equal(a.get_conserved(), w0)
        assert a.step_dt(1, dt) == 0 and np.array_equal(a.get_conserved(), w1)
    a.set_state(p.prim)
    assert a.step(1) == 0                     # a pass of its own: the same formula on the same numbers
    assert a.stats()["dt_last"] == pytest.approx(dt, rel=1e-14)
    a.set_state(p.prim)                       # with it again
    assert a.step(1) == 0 and a.stats()["dt_last"] == dt
    assert np.array_equal(a.get_conserved(), w1)
    # a fixed dt never needs it
    p.dt_fixed = dt
    f = m2c.Sim(m2c.config_for(p), p.prim)
    assert f.step(1) == 0 and f.stats()["dt_last"] == dt
    assert np.array_equal(f.get_conserved(), w1)
    if p.eos is None:
        b = m2c.Batch([m2c.config_for(p, tile=f.tile())] * 2, [p.prim] * 2)
        assert b.step(1) == 0 and b.stats(1)["dt_last"] == dt
        b.set_state(1, p.prim)
        assert b.step(1) == 0 and b.stats(1)["dt_last"] == dt
