"""The flight step's short forms against the general ones (host build of the
device header): the slab filter never passes a flight that may leave, and the
staged tables' band search gives the general search's band, majorant and
edge, at the edges themselves, for NaN and infinity, in both precisions."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2509_15377_amd", "csrc")


@pytest.fixture(scope="module")
def results(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc")
    exe = str(tmp_path_factory.mktemp("ff") / "flight_filters")
    subprocess.run([hipcc, "-x", "hip", "--offload-host-only", "-std=c++17", "-O2", "-ffp-contract=off", "-I", CSRC,
                    os.path.join(ROOT, "tests", "flight_filters.cpp"), "-o", exe],
                   check=True, capture_output=True)
    out = subprocess.run([exe], check=True, capture_output=True, text=True, timeout=120).stdout
    return {name: tuple(int(v) for v in rest) for name, *rest in (line.split() for line in out.splitlines())}


@pytest.mark.parametrize("check", ["slab_f64", "slab_f32", "bands_f64", "bands_f32"])
def test_short_form_agrees(results, check):
    n, used, bad = results[check]
    assert n > 10000 and used > n // 10
    assert bad == 0
