"""A run beside another kernel that holds half of the CUs: the same bits, and
no more than a run on half of the device takes.  Half of the waves take twice
as long; twice that again is allowed for.  (Rules that went by the grid's waves
kept every wave at a few electrons here: 238 ms where the free device takes 16
and half of it 24.)"""
import ctypes as C
import os
import shutil
import subprocess
import time

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def hold(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    so = str(tmp_path_factory.mktemp("hold") / "hold_cus.so")
    subprocess.run([hipcc, "--offload-arch=gfx950", "-O2", "-shared", "-fPIC", "-Xclang", "-target-feature",
                    "-Xclang", "-packed-fp32-ops", os.path.join(ROOT, "tests", "hold_cus.hip"), "-o", so],
                   check=True, capture_output=True)
    import torch  # noqa: F401  (its HIP runtime first: the libraries then bind to the same one)
    fn = C.CDLL(so).hold_cus
    fn.argtypes = [C.c_int, C.c_int, C.c_double, C.c_void_p, C.c_void_p]
    return fn


@pytest.mark.parametrize("precision", [0, 1])
def test_half_of_the_cus_held(hold, precision):
    import torch

    from paper_2509_15377_amd import avm, workloads as W
    w = W.argon(1000, band_bins=100)
    g, f = avm.Gas(w.gas, 0), avm.Field(w.field, 0)
    side, stream = torch.cuda.Stream(), torch.cuda.Stream()
    out = torch.zeros(256, dtype=torch.int32, device="cuda:0")
    r = avm.Run(g, f, w.primaries, w.n_aval, seed=w.seed, precision=precision, majorant=avm.BANDED,
                mode=avm.BATCHED, capacity=8_000_000, band_lookahead=1.0, stream=stream, timeout_s=20.0)

    def timed():
        t = time.perf_counter()
        r.execute()
        r.sync()
        return time.perf_counter() - t

    def result():
        ep = r.endpoints()
        return ep[np.lexsort((ep["eid"], ep["aval"]))].tobytes()
    timed()
    free = min(timed() for _ in range(3))
    ref = result()
    torch.cuda.synchronize()
    assert hold(0, 128, 400.0, out.data_ptr(), side.cuda_stream) == 0
    time.sleep(0.005)
    half = min(timed() for _ in range(2))
    beside = not side.query()
    torch.cuda.synchronize()
    print(f"free {1e3 * free:.1f} ms, half of the CUs held {1e3 * half:.1f} ms", flush=True)
    assert beside and half < 4.0 * free
    assert result() == ref
    r.close()
