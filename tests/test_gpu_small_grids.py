"""Small grids: the default number of planes per stage block (FP64: few planes,
so that the blocks of a small grid spread over the chip) against blocks of 8
planes, for single contexts and batches; mixed precision keeps 8 (needs an
MI355X)."""
from __future__ import annotations

import numpy as np
import pytest

import workloads as W
from tests.parity import conserved_errors

pytestmark = pytest.mark.gpu

# Planes per block change which code computes a block's lowest z-face (the
# prologue of its march or the loop), the same formulas in another place: in
# FP64 the runs differ by roundings that grow over the steps (1e-12, 1000
# times below the oracle bar); in mixed precision the blocks are the same, and
# so are the results.
TOL = {0: 1e-12, 1: 0.0}


@pytest.fixture(scope="module")
def m2c():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2508_16387_amd as m
    m.lib()
    return m


def _same(wa, wb, prim, chi, p, tol):
    e = conserved_errors(wa, wb, prim, p.gamma, p.pc, chi, min(p.dx()))
    assert max(e.values()) <= tol, e


# one plane, a few planes, the last size below 8 planes and the first at 8
@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("dims", [(17, 16, 3), (33, 31, 30), (64, 60, 62), (96, 90, 60), (100, 100, 110)])
def test_default_planes(m2c, dims, prec):
    p = W.shock_bubble(3, nxyz=dims, radius=0.2, p_shock=1e9, shock_x=0.25)
    a = m2c.Sim(m2c.config_for(p, precision=prec), p.prim)
    b = m2c.Sim(m2c.config_for(p, precision=prec, tile=(16, 15, 8)), p.prim)
    assert a.tile()[2] < 8 or prec == 1 or dims[2] > 100
    assert a.step(6) == 0 and b.step(6) == 0
    prim, chi = b.get_state()
    assert np.array_equal(a.get_state()[1], chi)
    _same(a.get_conserved(), b.get_conserved(), prim, chi, p, TOL[prec])


# a batch small enough for few planes, one whose 32x7 cover is too wasteful
@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("dims", [[(40, 33, 21), (24, 30, 40)], [(17, 17, 9)], [(64, 64, 48)] * 4])
def test_default_batch_tile(m2c, dims, prec):
    ps = [W.shock_bubble(5 + k, nxyz=d, radius=0.2, p_shock=1e9, shock_x=0.25) for k, d in enumerate(dims)]
    b = m2c.Batch([m2c.config_for(p, precision=prec) for p in ps], [p.prim for p in ps])
    assert b.step(5) == 0
    for k, p in enumerate(ps):
        s = m2c.Sim(m2c.config_for(p, precision=prec, tile=(16, 16, 8)), p.prim)
        assert s.step(5) == 0
        prim, chi = s.get_state()
        assert np.array_equal(b.get_state(k)[1], chi)
        _same(b.get_conserved(k), s.get_conserved(), prim, chi, p, TOL[prec])
