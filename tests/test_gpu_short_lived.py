"""Many electrons of few flights, where the claims are most of the run: the
bits of the plain mode at the numbers where the blocks' and the waves' shares
change, and no more time than the claims take (30000 electrons: 130 us of
kernel time; one atomic for each of 4096 waves and four electrons a wave made
it 420; 100000: 180 and 500.  The bar is twice the time)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _run(avm, g, f, prim, **kw):
    r = avm.Run(g, f, prim, prim.size, seed=3, majorant=avm.BANDED, band_lookahead=1.0, capacity=prim.size + 64,
                timeout_s=30.0, **kw)
    r.execute()
    r.sync()
    return r


def _case(n):
    from paper_2509_15377_amd import avm, workloads as W
    prim = W.primaries_at_rest(n, z=5e-6)
    prim["e"] = 5.0
    return avm.Gas(W.argon_like_gas(band_bins=100), 0), avm.Field(W.slab(1e-5, 2e4), 0), prim


@pytest.mark.parametrize("n", [1, 2, 255, 256, 257, 1023, 1024, 1025, 4095, 4097, 16383, 16385, 262144, 300000])
def test_shares(n):
    from paper_2509_15377_amd import avm
    g, f, prim = _case(n)
    out = []
    for mode, kw in ((avm.PLAIN, {}), (avm.BATCHED, {}), (avm.BATCHED, {"flights_per_pass": 1})):
        print(n, mode, kw, flush=True)
        r = _run(avm, g, f, prim, mode=mode, **kw)
        ep = r.endpoints()
        out.append(ep[np.lexsort((ep["eid"], ep["aval"]))].tobytes())
        r.close()
    assert len(out[0]) == n * avm.ENDPOINT_DTYPE.itemsize
    assert out[1] == out[0] and out[2] == out[0]


@pytest.mark.parametrize("n,limit_us", [(30000, 260.0), (100000, 360.0)])
def test_time(n, limit_us):
    from paper_2509_15377_amd import avm
    g, f, prim = _case(n)
    r = _run(avm, g, f, prim, mode=avm.BATCHED)
    us = []
    for _ in range(8):
        r.execute()
        r.sync()
        us.append(1e3 * r.timing()[0])
    r.close()
    print(f"{n} electrons: {min(us):.0f} us", flush=True)
    assert min(us) < limit_us
