"""The rules by which waves hand secondaries on, for the numbers of waves that
may have started: when all of them carry electrons they keep their own, when
few do they spread."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2509_15377_amd", "csrc")


def test_rules(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc")
    exe = str(tmp_path / "wave_load")
    subprocess.run([hipcc, "-x", "hip", "--offload-host-only", "-std=c++17", "-O2", "-I", CSRC, "-I",
                    os.path.join(ROOT, "include"), os.path.join(ROOT, "tests", "wave_load.cpp"), "-o", exe],
                   check=True, capture_output=True)
    rows = subprocess.run([exe], check=True, capture_output=True, text=True, timeout=60).stdout.splitlines()
    assert len(rows) == 6 * 17
    for waves, busy, full, spare, spread, spread_filled in (map(int, r.split()) for r in rows):
        assert full == (8 * busy > 7 * waves) and spare == (8 * busy < 7 * waves)
        assert spread == (2 * busy <= waves) and spread_filled == (8 * busy <= waves)
        if busy == waves:
            assert full and not spare and not spread and not spread_filled
        if busy == 0:
            assert spare and spread and spread_filled
