"""Length of a pass for every number of flights that a caller may ask for: at
least one flight, as many as asked for (half with a long queue, four times as
many in a sparse wave), up to the bound above which longer ones are cut."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2509_15377_amd", "csrc")
MOST = 1 << 28


def test_pass_lengths(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc")
    exe = str(tmp_path / "pass_lengths")
    subprocess.run([hipcc, "-x", "hip", "--offload-host-only", "-std=c++17", "-O2", "-I", CSRC, "-I",
                    os.path.join(ROOT, "include"), os.path.join(ROOT, "tests", "pass_lengths.cpp"), "-o", exe],
                   check=True, capture_output=True)
    rows = subprocess.run([exe], check=True, capture_output=True, text=True, timeout=60).stdout.splitlines()
    assert len(rows) == 24
    for n, long_queue, flights, dense, sparse in (map(int, r.split()) for r in rows):
        want = min(n, MOST)
        want = (want + 1) // 2 if long_queue else want
        assert (flights, dense, sparse) == (want, want, 4 * want)
