"""A step that fails at its interface faces in the middle of one call of many
steps: the steps before it are closed exactly as when each is a call of its
own (needs an MI355X)."""
from __future__ import annotations

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def m2c():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2508_16387_amd as m
    m.lib()
    return m


def _pulled_apart(n, boost, jump, at):
    """An air bubble in a very stiff liquid (p_c 1e11 Pa) that moves at
    `boost`; the liquid beyond x = at moves away at `jump`, and when the
    rarefaction from there reaches the bubble, the liquid leaves its surface
    faster than the air can follow: no star pressure above 0."""
    x, y, z = ((np.arange(k) + 0.5) / k for k in n)
    Z, Y, X = np.meshgrid(z, y, x, indexing="ij")
    phi = np.sqrt((X - 0.5) ** 2 + (Y - 0.5) ** 2 + (Z - 0.5) ** 2) - 0.3
    f = np.zeros((6, n[2], n[1], n[0]))
    f[0] = np.where(phi >= 0, 1000.0, 1.0)
    f[1] = boost + np.where(X > at, jump, 0.0)
    f[4] = 1e5
    f[5] = phi
    return W.Problem("pulled_apart", n, (0.0, 0.0, 0.0), (1.0, 1.0, 1.0), gamma=(6.12, 1.4), pc=(1e11, 0.0),
                     cfl=0.4, prim=f)


# Forward Euler has one interface launch per step, the one that also opens it,
# so the failure is in that launch; with two stages it may be in either.
# rebuilt: whether the failing step's queue is a new one (the step before
# flipped cells).
CASES = [((32, 28, 24), 0.0, 3000.0, 0.86, False), ((32, 28, 24), 2000.0, 3000.0, 0.86, False),
         ((32, 28, 24), 2000.0, 3000.0, 0.95, True), ((32, 28, 24), 2000.0, 6000.0, 0.9, True),
         ((96, 90, 80), 2000.0, 6000.0, 0.86, None)]


@pytest.mark.parametrize("rk", [1, 2])
@pytest.mark.parametrize("n,boost,jump,at,rebuilt", CASES)
def test_steps_before_a_failing_one_are_closed(m2c, n, boost, jump, at, rebuilt, rk):
    p = _pulled_apart(n, boost, jump, at)
    cfg = m2c.config_for(p, rk_order=rk)
    one = m2c.Sim(cfg, p.prim)
    rc, done, flips = 0, 0, [0]
    while rc == 0 and done < 200:
        before = one.stats()
        state = one.get_conserved()
        rc = one.step(1, check=False)
        done += rc == 0
        flips.append(one.stats()["flips"])
    assert rc == m2c.M2C_ERR_RIEMANN and done > 5
    if rebuilt is not None and rk == 1:
        assert (flips[-2] != flips[-3]) == rebuilt
    where = one.stats()["err_cell"]
    assert np.array_equal(one.get_conserved(), state)
    for first in (0, 3):
        many = m2c.Sim(cfg, p.prim)
        assert many.step(first) == 0
        assert many.step(done + 7 - first, check=False) == m2c.M2C_ERR_RIEMANN
        st = many.stats()
        for k in ("steps", "t", "dt_last", "flips", "riemann_solves", "orphans"):
            assert st[k] == before[k], (k, st[k], before[k])
        assert st["steps"] == done and st["err_code"] == m2c.M2C_ERR_RIEMANN
        assert f"step {done + 1} failed" in many.last_error()
        if rk == 1:
            assert st["err_cell"] == where
        assert np.array_equal(many.get_conserved(), state)
        # and it goes on from there: the same step fails again
        assert many.step(2, check=False) == m2c.M2C_ERR_RIEMANN
        assert many.stats()["steps"] == done and np.array_equal(many.get_conserved(), state)


def test_queue_overflow_is_the_only_error(m2c):
    """More interface faces than the queue holds, some of them without a star
    pressure: the status is the overflow, and no step is counted."""
    n = (64, 64, 32)                                    # 131072 cells, as many queue entries
    f = np.zeros((6, n[2], n[1], n[0]))
    k, j, i = np.indices((n[2], n[1], n[0]))
    f[5] = np.where((i + j + k) % 2, 1.0, -1.0)         # every face
    f[0] = np.where(f[5] >= 0, 1000.0, 1.0)
    f[1] = np.where(i >= n[0] // 2, 1e6, 0.0)
    f[4] = 1e5
    p = W.Problem("checkerboard", n, (0.0, 0.0, 0.0), (1.0, 1.0, 0.5), gamma=(6.12, 1.4), pc=(3.43e8, 0.0), prim=f)
    s = m2c.Sim(m2c.config_for(p), f)
    w = s.get_conserved()
    for _ in range(3):
        assert s.step(4, check=False) == m2c.M2C_ERR_NOMEM
        assert s.stats()["steps"] == 0 and s.stats()["riemann_solves"] == 0
        assert np.array_equal(s.get_conserved(), w)
