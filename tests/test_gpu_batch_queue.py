"""The batch's kept and rebuilt interface queues: runs whose interface moves
beside runs whose queue is kept from step to step, through replaced states and
a failing run, against single contexts (needs an MI355X)."""
from __future__ import annotations

import numpy as np
import pytest

import workloads as W
from tests.test_gpu_batch import assert_batch_matches, m2c  # noqa: F401

pytestmark = pytest.mark.gpu


def _problems():
    """A tube whose interface moves, bubbles before the shock reaches them (no
    flips), one with many faces, and a single-material box (an empty queue)."""
    return [W.shock_tube_1d(0, nx=700), W.shock_bubble(1, nxyz=(20, 18, 17), radius=0.2),
            W.shock_bubble(2, nxyz=(48, 40, 36), radius=0.4, p_shock=1e9, shock_x=0.08),
            W.periodic_box(3, n=(12, 10, 9))]


@pytest.mark.parametrize("split", [(12,), (1, 11), (5, 1, 6)])
def test_kept_and_rebuilt_queues(m2c, split):  # noqa: F811
    ps = _problems()
    b = m2c.Batch([m2c.config_for(p) for p in ps], [p.prim for p in ps])
    sims = [m2c.Sim(m2c.config_for(p), p.prim) for p in ps]
    for n in split:
        assert b.step(n) == 0
        for k, s in enumerate(sims):
            assert s.step(n) == 0
            assert_batch_matches(b, k, s, ps[k])
            sb, ss = b.stats(k), s.stats()
            assert all(sb[q] == ss[q] for q in ("steps", "flips", "riemann_solves", "iface_faces_last")), (k, sb, ss)
    assert b.stats(0)["flips"] > 0 and b.stats(1)["flips"] == 0
    # a replaced state starts from its own queue
    q = W.shock_bubble(7, nxyz=(20, 18, 17), radius=0.3)
    b.set_state(1, q.prim)
    sims[1].set_state(q.prim)
    assert b.step(3) == 0 and sims[1].step(3) == 0
    assert_batch_matches(b, 1, sims[1], q)
