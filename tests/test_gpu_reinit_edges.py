"""Level-set reinitialization at the edges of its decomposition (a block's 256
columns and 4 planes, one-cell axes, periodic wraps within a block), against
the oracle (needs an MI355X)."""
from __future__ import annotations

import numpy as np
import pytest

from oracle import reinit as RI
from tests.test_gpu_reinit import m2c, run_gpu  # noqa: F401

pytestmark = pytest.mark.gpu


# The library forms the same Jacobi iterates in FP64: 1e-12 of max|phi_0|, as
# in the other reinitialization tests.
@pytest.mark.parametrize("bc", [(0, 0, 1, 1, 0, 1), (2, 2, 2, 2, 2, 2)])
@pytest.mark.parametrize("band", [0.0, 0.3])
@pytest.mark.parametrize("dims", [(7, 1, 1), (1, 1, 9), (1, 300, 2), (257, 1, 1), (16, 16, 4), (5, 3, 5), (51, 5, 8),
                                  (65, 63, 3), (2, 2, 2)])
def test_reinit_edges(m2c, dims, band, bc):  # noqa: F811
    nx, ny, nz = dims
    rng = np.random.default_rng(nx * 1000 + ny * 10 + nz)
    x, y, z = (np.linspace(-1.0, 1.0, n) if n > 1 else np.zeros(1) for n in dims)
    phi0 = (0.4 * np.sin(3 * x)[None, None, :] + 0.3 * np.cos(2 * y)[None, :, None] - 0.2 * np.sin(4 * z)[:, None, None]
            + 0.02 * rng.standard_normal((nz, ny, nx)))
    h = tuple(2.0 / n for n in dims)
    got = run_gpu(m2c, phi0, h, bc, 5, band)
    ref = RI.reinit(phi0, h, bc, 5, band=band)
    assert np.max(np.abs(got - ref)) <= 1e-12 * np.max(np.abs(phi0))
