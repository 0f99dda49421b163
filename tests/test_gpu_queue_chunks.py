"""The interface queue of grids above 4096 compaction blocks, which a launch
block takes several of at a time, by words and by bytes, alone and in a batch
(needs an MI355X)."""
from __future__ import annotations

import numpy as np
import pytest

import workloads as W
from tests.test_gpu_batch import assert_batch_matches
from tests.test_gpu_queue_launch import m2c  # noqa: F401
from tests.test_gpu_queue_units import _faces

pytestmark = pytest.mark.gpu


def _problem(n):
    """Two bubbles, a flat surface across z and one scattered cell in about
    9000, moving along x."""
    nx, ny, nz = n
    z, y, x = (np.arange(nz) + 0.5) / nz, (np.arange(ny) + 0.5) / ny, (np.arange(nx) + 0.5) / nx
    phi = np.full((nz, ny, nx), 1.0)
    for c, r in (((0.3, 0.4, 0.2), 0.1), ((0.6, 0.7, 0.8), 0.15)):
        d = np.sqrt((z[:, None, None] - c[2]) ** 2 + (y[:, None] - c[1]) ** 2 + (x - c[0]) ** 2) - r
        phi = np.minimum(phi, d)
    phi = np.minimum(phi, 0.97 - z[:, None, None])
    phi.reshape(-1)[::9001] = -0.3 / nx
    f = np.zeros((6, nz, ny, nx))
    f[5] = phi
    f[0] = np.where(phi >= 0, 1000.0, 1.0)
    f[1] = 3000.0
    f[4] = 1e5
    return W.Problem("chunks", n, (0.0, 0.0, 0.0), (1.0, 1.0, 1.0), gamma=(W.WATER[0], W.AIR[0]),
                     pc=(W.WATER[1], W.AIR[1]), cfl=0.4, prim=f)


@pytest.mark.parametrize("n", [(256, 256, 257), (259, 257, 255), (512, 260, 255)])
def test_queue_by_chunks(m2c, n):  # noqa: F811
    p = _problem(n)
    tile = (16, 15, 8)
    s = m2c.Sim(m2c.config_for(p, tile=tile), p.prim)
    small = W.shock_bubble(1, nxyz=(20, 18, 17), radius=0.2)
    b = m2c.Batch([m2c.config_for(q, tile=tile) for q in (small, p)], [small.prim, p.prim])
    solves = 0
    for k in range(3):
        faces = _faces(s.get_state()[1])
        assert k != 1 or np.array_equal(s.interface_faces(), faces)
        assert s.step(1) == 0 and b.step(1) == 0
        st, sb = s.stats(), b.stats(1)
        solves += 2 * len(faces)
        assert st["iface_faces_last"] == sb["iface_faces_last"] == len(faces)
        assert st["riemann_solves"] == sb["riemann_solves"] == solves
    assert np.array_equal(s.interface_faces(), _faces(s.get_state()[1]))
    assert st["flips"] == sb["flips"] > 0
    assert_batch_matches(b, 1, s, p)
