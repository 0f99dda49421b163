"""A run of a batch that fails, beside runs whose queues are kept and rebuilt:
its own state, counters and next steps, and its neighbours', against single
contexts (needs an MI355X)."""
from __future__ import annotations

import numpy as np
import pytest

import workloads as W
from tests.test_gpu_batch import assert_batch_matches, m2c  # noqa: F401
from tests.test_gpu_failing_step import _pulled_apart

pytestmark = pytest.mark.gpu

COUNTERS = ("steps", "flips", "riemann_solves", "orphans", "err_code")


def _problems():
    """A bubble whose surface is pulled apart after some steps, with cells
    flipping (0) and not (1); a tube far above the stability limit (2); a tube
    whose interface moves (3) and a bubble at rest (4)."""
    unstable = W.shock_tube_1d(3, nx=200)
    unstable.cfl = 5.0
    return [_pulled_apart((32, 28, 24), 2000.0, 3000.0, 0.95), _pulled_apart((32, 28, 24), 0.0, 3000.0, 0.86), unstable,
            W.shock_tube_1d(0, nx=700), W.shock_bubble(1, nxyz=(20, 18, 17), radius=0.2)]


@pytest.mark.parametrize("split", [(60, 3, 1), (7, 1, 50, 2)])
def test_failing_runs(m2c, split):  # noqa: F811
    ps, tile = _problems(), (16, 15, 8)
    cfgs = [m2c.config_for(p, tile=tile) for p in ps]
    b = m2c.Batch(cfgs, [p.prim for p in ps])
    sims = [m2c.Sim(c, p.prim) for c, p in zip(cfgs, ps)]

    def step(n):
        rcs = [s.step(n, check=False) for s in sims]
        assert b.step(n, check=False) == next((rc for rc in rcs if rc != 0), 0)
        for k, s in enumerate(sims):
            sb, ss = b.stats(k), s.stats()
            assert all(sb[q] == ss[q] for q in COUNTERS), (k, n, sb, ss)
            assert sb["t"] == pytest.approx(ss["t"], rel=1e-12)
            assert_batch_matches(b, k, s, ps[k])
            if rcs[k] == 0:
                assert sb["iface_faces_last"] == ss["iface_faces_last"], (k, n)
        return rcs

    for n in split:
        rcs = step(n)
    assert rcs[0] == rcs[1] == m2c.M2C_ERR_RIEMANN and rcs[2] != 0 and rcs[3] == rcs[4] == 0
    # a failed run goes on from a new state, on its own queue
    q = W.shock_bubble(9, nxyz=(32, 28, 24), radius=0.3)
    for k in (0, 1):
        f = np.array(q.prim)
        f[0] = np.where(f[5] >= 0, 1000.0, 1.0)
        f[4] = 1e5
        f[1:4] = 0.0
        f[1] = 2000.0 if k else 0.0
        b.set_state(k, f)
        sims[k].set_state(f)
    for n in (1, 2, 5):
        rcs = step(n)
        assert rcs[0] == rcs[1] == rcs[3] == rcs[4] == 0 and rcs[2] != 0
