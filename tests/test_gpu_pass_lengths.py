"""Passes longer than any electron's life ("until it stops"): the same bits
as with the default pass, for runs that start sparse and that fill waves."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("n", [1, 40])
def test_very_long_passes(n, precision):
    from paper_2509_15377_amd import avm, workloads as W
    w = W.argon(n, band_bins=100)
    w.field = W.slab(60e-4, 45e3)
    g, f = avm.Gas(w.gas, 0), avm.Field(w.field, 0)
    ref = None
    for fpp in (0, 1 << 28, 1 << 29, 1 << 30, 2 ** 31 - 1):
        print(n, precision, fpp, flush=True)
        r = avm.Run(g, f, w.primaries, n, seed=4, precision=precision, majorant=avm.BANDED, mode=avm.BATCHED,
                    capacity=1 << 19, flights_per_pass=fpp, band_lookahead=1.0, timeout_s=30.0)
        r.execute()
        r.sync()
        ep = r.endpoints()
        r.close()
        ep = ep[np.lexsort((ep["eid"], ep["aval"]))].tobytes()
        ref = ref or ep
        assert ep == ref, fpp
