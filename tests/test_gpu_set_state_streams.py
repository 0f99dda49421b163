"""A state is set when the call returns: nothing of it is pending on the
context's stream, and the next step may run on another (needs an MI355X)."""
from __future__ import annotations

import numpy as np
import pytest

import workloads as W
from tests.test_gpu_batch import m2c  # noqa: F401

pytestmark = pytest.mark.gpu


def test_set_on_one_stream_step_on_another(m2c):  # noqa: F811
    import torch
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    ps = [W.shock_tube_1d(k, nx=300) for k in range(3)]
    ref = []
    for p in ps:
        s = m2c.Sim(m2c.config_for(p), p.prim)
        assert s.step(2) == 0
        ref.append((s.stats()["dt_last"], s.get_conserved()))
    bad = np.array(ps[0].prim)
    bad[4].flat[-1] = -1e12
    s = m2c.Sim(m2c.config_for(ps[0]))
    dev = [torch.from_numpy(p.prim).cuda() for p in ps]
    torch.cuda.synchronize()
    for rep in range(30):
        k = rep % 3
        s.set_stream(a if rep % 2 else b)
        if rep % 4 == 3:
            assert s.set_state(bad, check=False) == m2c.M2C_ERR_NONPHYSICAL
            assert (a if rep % 2 else b).query()
        if rep % 5:
            s.set_state_device(dev[k])
        else:
            s.set_state(ps[k].prim)
        assert (a if rep % 2 else b).query(), rep           # idle
        s.set_stream(b if rep % 2 else a)
        assert s.step(2) == 0
        assert s.stats()["dt_last"] == ref[k][0]
        assert np.array_equal(s.get_conserved(), ref[k][1])
