"""Register budget of the general-EOS point solver that dispatches over the
families without Mie-Grueneisen (compile-time, no GPU): two waves per SIMD, and
no more spilling than it was measured with."""
from __future__ import annotations

import os
import shutil
import subprocess

import pytest

from paper_2508_16387_amd import build as B
from tests.test_build_resources import HIPCC, _parse


def test_dispatch_without_mie_grueneisen(tmp_path):
    if not os.path.exists(HIPCC) and not shutil.which("hipcc"):
        pytest.skip("hipcc not available")
    src = "k_riemann_eos.hip"
    p = subprocess.run([HIPCC, *B.flags_for(src), "-c", os.path.join(B.CSRC, src), "-o", str(tmp_path / "o.o"),
                        "-Rpass-analysis=kernel-resource-usage"], capture_output=True, text=True)
    assert p.returncode == 0, p.stderr[-2000:]
    ks = {n: r for n, r in _parse(p.stderr).items() if "k_riemann_eosILin2ELin1E" in n}
    assert len(ks) == 1, sorted(ks)
    for n, r in ks.items():
        assert r["occupancy"] >= 2 and r["scratch"] <= 164, (n, r)
