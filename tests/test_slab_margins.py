"""The slab filter with the margins of the library's own fields never passes a
flight that may leave: flights that end or turn close to a plane (host build of
the device header)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2509_15377_amd", "csrc")


def test_filter_is_conservative(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc")
    exe = str(tmp_path / "slab_margins")
    subprocess.run([hipcc, "-x", "hip", "--offload-host-only", "-std=c++17", "-O2", "-ffp-contract=off", "-I", CSRC,
                    os.path.join(ROOT, "tests", "slab_margins.cpp"), "-o", exe], check=True, capture_output=True)
    rows = subprocess.run([exe], check=True, capture_output=True, text=True, timeout=120).stdout.split("\n")
    seen = {name: tuple(map(int, rest)) for name, *rest in (r.split() for r in rows if r)}
    for name in ("f64", "f32"):
        n, clear, bad = seen[name]
        assert n == 2000000 and clear > n // 10
        assert bad == 0
