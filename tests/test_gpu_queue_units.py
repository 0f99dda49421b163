"""A rebuilt queue shared out in units of at most 256 faces, where an interface
lies in few compaction blocks: cell layers of z, whole blocks of faces, counts
beside a multiple of 256 (needs an MI355X)."""
from __future__ import annotations

import numpy as np
import pytest

import workloads as W
from tests.test_gpu_queue_launch import m2c  # noqa: F401

pytestmark = pytest.mark.gpu


def _faces(chi):
    """Interface faces 3 c + d of the ids, ascending (no periodic axis)."""
    nz, ny, nx = chi.shape
    c = np.arange(chi.size).reshape(chi.shape)
    f = [3 * c[:, :, :-1][chi[:, :, 1:] != chi[:, :, :-1]], 3 * c[:, :-1][chi[:, 1:] != chi[:, :-1]] + 1,
         3 * c[:-1][chi[1:] != chi[:-1]] + 2]
    return np.sort(np.concatenate(f))


def _problem(n, layers, holes, u):
    """Layers of air in water across z (one cell thick each, so 2 faces per
    cell of a layer), `holes` cells of them water again, and a column of air
    whose side moves along x, so that cells flip; uniform pressure and
    velocity, a moving two-material contact."""
    nx, ny, nz = n
    k, j, i = np.indices((nz, ny, nx))
    air = np.isin(k, layers)
    air.reshape(-1)[np.flatnonzero(air.reshape(-1))[:holes]] = False
    x = (i + 0.5) / nx
    phi = np.where(air, -0.5 / nz, np.where(x < 0.2, x - 0.2, 0.5 / nz))
    f = np.zeros((6, nz, ny, nx))
    f[5] = phi
    f[0] = np.where(phi >= 0, 1000.0, 1.0)
    f[1] = u
    f[4] = 1e5
    return W.Problem("layers", n, (0.0, 0.0, 0.0), (1.0, ny / nx, nz / nx), gamma=(W.WATER[0], W.AIR[0]),
                     pc=(W.WATER[1], W.AIR[1]), cfl=0.4, prim=f)


# The same step solved with the queue written by the opening launch (at most
# 512 compaction blocks) and with the queue listed before it, in a launch of
# its own, and then kept: the same solves, so the same bits.
@pytest.mark.parametrize("n,layers,holes", [((64, 64, 32), [9, 20], 0), ((64, 64, 32), [9, 10, 11], 1),
                                            ((17, 19, 23), [5, 11], 7), ((16, 16, 8), [3], 0), ((16, 16, 8), [3], 1),
                                            ((128, 128, 128), [40, 90], 300), ((130, 126, 128), [64], 0)])
def test_units_cover_the_queue(m2c, n, layers, holes):  # noqa: F811
    p = _problem(n, layers, holes, 3000.0)       # 1.3 cells in 8 steps
    cfg = m2c.config_for(p)
    a, b = m2c.Sim(cfg, p.prim), m2c.Sim(cfg, p.prim)
    flips = 0
    for _ in range(8):
        chi = b.get_state()[1]
        assert np.array_equal(b.interface_faces(), _faces(chi))     # b's queue: a launch of its own
        assert a.step(1) == 0 and b.step(1) == 0
        sa, sb = a.stats(), b.stats()
        assert sa["iface_faces_last"] == len(_faces(chi))
        for q in ("riemann_solves", "newton_iters", "bisection_fallbacks", "flips", "dt_last"):
            assert sa[q] == sb[q], q
        assert np.array_equal(a.get_conserved(), b.get_conserved())
        flips = sa["flips"]
    c = m2c.Sim(cfg, p.prim)
    assert c.step(8) == 0 and np.array_equal(c.get_conserved(), a.get_conserved())
    assert flips > 0
