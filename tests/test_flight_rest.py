"""The collision decision of an electron at rest, where the edge of channel
0's window is as near as its energy: in FP32-mixed it is taken as in FP64, in
gases of one channel and of several (host build of the device header)."""
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
    exe = str(tmp_path_factory.mktemp("rest") / "flight_rest")
    subprocess.run([hipcc, "-x", "hip", "--offload-host-only", "-std=c++17", "-O2", "-ffp-contract=off", "-I", CSRC,
                    os.path.join(ROOT, "tests", "flight_rest.cpp"), "-o", exe],
                   check=True, capture_output=True)
    out = subprocess.run([exe], check=True, capture_output=True, text=True, timeout=120).stdout
    return {name: tuple(int(v) for v in rest) for name, *rest in (line.split() for line in out.splitlines())}


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("majorant", ["banded", "global"])
@pytest.mark.parametrize("tables", ["global", "staged"])
@pytest.mark.parametrize("gas", ["one", "two", "three", "late"])
def test_decision_at_rest(results, gas, tables, majorant, precision):
    n, real, bad = results[f"{gas}-{tables}-{majorant}-{precision}"]
    assert n == 4000 and real > n // 4
    assert bad == 0
