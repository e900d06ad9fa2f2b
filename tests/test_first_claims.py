"""First claims of the persistent kernel's blocks and waves (host build): no
entry is left without a lane or taken twice, whatever the number of entries
and of blocks, and together the blocks claim every entry their lanes can hold."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2509_15377_amd", "csrc")


def test_every_claimed_entry_has_one_lane(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc")
    exe = str(tmp_path / "first_claims")
    subprocess.run([hipcc, "-x", "hip", "--offload-host-only", "-std=c++17", "-O2", "-I", CSRC, "-I",
                    os.path.join(ROOT, "include"), os.path.join(ROOT, "tests", "first_claims.cpp"), "-o", exe],
                   check=True, capture_output=True)
    rows = subprocess.run([exe], check=True, capture_output=True, text=True, timeout=60).stdout.splitlines()
    assert len(rows) == 300
    for n, blocks, claimed, bad, used in (map(int, r.split()) for r in rows):
        assert bad == 0, (n, blocks)
        assert claimed == min(n, blocks * 1024), (n, blocks)
        # a wave per electron at most, and no more than one SIMD's share needs
        assert used <= min(n, 16 * blocks)
