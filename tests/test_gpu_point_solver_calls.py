"""The point solvers' calls: the failure flag over threads and streams, and
the grouping of general-EOS sets at its block edges (needs an MI355X)."""
from __future__ import annotations

import threading

import numpy as np
import pytest
import torch

import workloads as W
from tests.test_gpu_riemann_eos import TOL_EOS, _compare, _gpu, m2c  # noqa: F401

pytestmark = pytest.mark.gpu


def _sg(n, vacuum_at=None):
    inp = torch.tensor([[1000.0], [0.0], [1e7], [1.2], [0.0], [1e5]], dtype=torch.float64).repeat(1, n).cuda()
    inp[2] *= torch.linspace(1.0, 50.0, n, dtype=torch.float64, device="cuda")
    eos = torch.tensor([[4.4], [6e8], [1.4], [0.0]], dtype=torch.float64).repeat(1, n).cuda()
    if vacuum_at is not None:
        inp[:, vacuum_at] = torch.tensor([1.2, -1e5, 1e5, 1.2, 1e5, 1e5], dtype=torch.float64)
        eos[:, vacuum_at] = torch.tensor([1.4, 0.0, 1.4, 0.0], dtype=torch.float64)
    return inp, eos


def test_failure_flag_over_threads_and_streams(m2c):  # noqa: F811
    bad = []

    def run(k):
        s = torch.cuda.Stream()
        n = 64 * (k + 1) + k
        sets = [_sg(n), _sg(n, vacuum_at=n // 2)]
        torch.cuda.synchronize()
        for rep in range(20):
            v = (rep + k) % 2
            out, it, rc = m2c.riemann_solve(*sets[v], stream=s.cuda_stream)
            s.synchronize()
            n0 = int((it == 0).sum())
            if rc != (m2c.M2C_ERR_RIEMANN if v else m2c.M2C_OK) or n0 != v:
                bad.append((k, rep, rc, n0))

    ts = [threading.Thread(target=run, args=(k,)) for k in range(4)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not bad, bad


FLUID = [("tnt", "water_sg"), ("water_sg", "air"), ("tnt", "tnt")]


@pytest.mark.parametrize("pairs", [FLUID, FLUID + [("air", "glass")]], ids=["no-mie-grueneisen", "all-families"])
def test_dispatch_and_grouping(m2c, pairs):  # noqa: F811
    """Sets of several family pairs against the oracle, and the same problems
    repeated to the edges of the grouping's blocks (2048 problems, at most
    256 blocks of 1024 threads): a copy has its problem's results bit for
    bit, also between problems with a material outside the table."""
    k = 61
    inp, mat, mats, _ = W.general_eos_problem_set(171, k, pairs=pairs)
    got, it, rc = _gpu(m2c, inp, mat, mats)
    e, ok = _compare(inp, mat, mats, got, it, "mixed")
    assert ok.sum() >= 45 and e.max() <= TOL_EOS, e.max(axis=1)
    for n in (1023, 2048, 2049, 4097, 256 * 2048 + 1):
        j = np.arange(n) % k
        m = mat[:, j].copy()
        m[n % 2, 5::977] = len(mats) if n % 2 else -1
        gotn, itn, rcn = _gpu(m2c, np.ascontiguousarray(inp[:, j]), m, mats)
        out = np.zeros(n, dtype=bool)
        out[5::977] = True
        assert rcn == m2c.M2C_ERR_RIEMANN
        assert np.isnan(gotn[:, out]).all() and (itn[out] == 0).all()
        assert np.array_equal(gotn[:, ~out], got[:, j[~out]], equal_nan=True)
        assert np.array_equal(itn[~out], it[j[~out]])
