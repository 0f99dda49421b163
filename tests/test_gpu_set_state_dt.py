"""The first time step after a state is set takes its CFL maximum from the
pass that sets it: against one taken from the conservative state, after a
rejected state, and in the batch (needs an MI355X)."""
from __future__ import annotations

import numpy as np
import pytest

import workloads as W
from tests.test_gpu_batch import m2c  # noqa: F401

pytestmark = pytest.mark.gpu


def _problems():
    return [W.shock_tube_1d(0, nx=37), W.shock_bubble(1, nxyz=(20, 18, 17), radius=0.2),
            W.shock_bubble(2, nxyz=(130, 97, 90), radius=0.3)]      # beyond 4096 blocks of 256 cells


@pytest.mark.parametrize("k", range(3))
def test_first_dt_and_rejected_state(m2c, k):  # noqa: F811
    p = _problems()[k]
    cfg = m2c.config_for(p)
    a, b = m2c.Sim(cfg, p.prim), m2c.Sim(cfg, p.prim)
    b.set_conserved(b.get_conserved())             # its maximum: a pass over the conservative state
    bad = np.array(p.prim)
    bad[4].flat[-1] = -1e12
    bad[1] += 1e4                                  # would raise the maximum
    batch = m2c.Batch([cfg], [p.prim])
    for n in (1, 2):
        assert a.step(n) == 0 and b.step(n) == 0 and batch.step(n) == 0
        # the same formula on the same numbers, at most contracted otherwise
        assert a.stats()["dt_last"] == pytest.approx(b.stats()["dt_last"], rel=1e-14)
        assert a.stats()["dt_last"] == batch.stats(0)["dt_last"]
        with pytest.raises(m2c.M2CError):
            a.set_state(bad)
        with pytest.raises(m2c.M2CError):
            batch.set_state(0, bad)
    a.set_state(p.prim)                            # nothing of the rejected state is left
    c = m2c.Sim(cfg, p.prim)
    assert a.step(1) == 0 and c.step(1) == 0
    assert a.stats()["dt_last"] == c.stats()["dt_last"]
