"""Mie-Grueneisen isentropes marched inside the compression branch (general-
EOS Riemann solver) at the ends of that march, against the oracle: states so
cold that the pressure nears its floor while the material is still
compressed (marches of hundreds to thousands of steps, and cavitation),
states just inside the branch whose march meets the branch point within a
step, and marches that end in the tension branches.  The bar and the error
measures are those of the other solver tests (TOL_EOS)."""
from __future__ import annotations

import numpy as np
import pytest

import workloads as W
from tests.test_gpu_riemann_eos import TOL_EOS, _compare, _gpu, m2c  # noqa: F401

pytestmark = pytest.mark.gpu


def _set(seed, n, eta, p, du):
    """Copper against tantalum: compressions eta and pressures p drawn from
    the ranges, closing or separating at du times the speed of sound."""
    rng = W.SplitMix64(seed)
    mats = [W.EOS_MATERIALS[m][:2] for m in ("copper", "tantalum")]
    inp, mat = np.zeros((6, n)), np.zeros((2, n), dtype=np.int32)
    for i in range(n):
        k = i % 2
        mat[:, i] = (k, 1 - k)
        for row, m in ((0, k), (3, 1 - k)):
            inp[row, i] = mats[m][1][0] / (1.0 - rng.uniform(*eta))
            inp[row + 2, i] = rng.uniform(*p)
        inp[4, i] = rng.uniform(*du) * 3414.0
    return inp, mat, [(f, list(q)) for f, q in mats]


CASES = {
    "cold_and_compressed": ((0.05, 0.057), (0.0, 5e8), (0.02, 0.06)),
    "at_the_branch_point": ((1e-8, 1e-4), (1e7, 1e9), (-0.02, 0.02)),
    "into_tension": ((0.002, 0.01), (5e8, 3e9), (0.0, 0.04)),
    "one_short_step": ((0.01, 0.05), (2e9, 3e9), (-1e-4, 1e-4)),
}


@pytest.mark.parametrize("name", list(CASES))
def test_compressed_march_matches_oracle(m2c, name):  # noqa: F811
    inp, mat, mats = _set(31 + list(CASES).index(name), 24, *CASES[name])
    got, it, rc = _gpu(m2c, inp, mat, mats)
    e, ok = _compare(inp, mat, mats, got, it, name)
    assert ok.sum() >= 4
    assert e.max() <= TOL_EOS, e.max(axis=1)
