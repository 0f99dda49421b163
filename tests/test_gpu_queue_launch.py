"""The interface queue of a step written by the first FIVER launch (up to 512
compaction blocks) and by a launch of its own (above), with a moving interface
so that it is rebuilt, against the faces the ids say and against each other
(needs an MI355X)."""
from __future__ import annotations

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

SEED = 0                 # 447 MPa: the interface crosses several cells in 60 steps


@pytest.fixture(scope="module")
def m2c():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2508_16387_amd as m
    m.lib()
    return m


def _near(m2c, nx, steps, half=200):
    """The tube's primitives within `half` cells of its middle, where the
    interface starts, and the interface faces before and after."""
    p = W.shock_tube_1d(SEED, nx=nx)
    s = m2c.Sim(m2c.config_for(p), p.prim)
    f0 = s.interface_faces()
    assert np.array_equal(f0, [3 * (nx // 2 - 1)])
    assert s.step(steps) == 0
    prim, chi = s.get_state()
    chi = chi[0, 0]
    at = np.flatnonzero(chi[1:] != chi[:-1])
    assert np.array_equal(s.interface_faces(), 3 * at)
    st = s.stats()
    assert st["flips"] > 0 and st["riemann_solves"] == 2 * steps and at[0] != nx // 2 - 1
    return prim[:, 0, 0, nx // 2 - half:nx // 2 + half], st


# 4096 cells per compaction block: 1, 2, 512 and 513 or more blocks.  In cell
# units the tube looks the same at every power-of-two size (dt scales with the
# cell width exactly), so the runs agree to FP64 rounding (1e-12 of the field)
# away from phi, which is a length.
@pytest.mark.parametrize("nx", [8192, 2 ** 21, 2 ** 22])
def test_rebuilt_queue_at_every_size(m2c, nx):
    ref, st0 = _near(m2c, 4096, 60)
    got, st = _near(m2c, nx, 60)
    assert st["flips"] == st0["flips"] and st["newton_iters"] == st0["newton_iters"]
    for v in range(5):
        assert np.max(np.abs(got[v] - ref[v])) <= 1e-12 * max(np.max(np.abs(ref[v])), 1e-30)
