"""Waves that carry few electrons (random numbers drawn ahead by all lanes,
secondaries spread over idle waves): the batched run equals the plain one bit
for bit at the electron counts where the split of the draws changes, in both
precisions, for passes shorter and longer than the draws."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _sorted(ep):
    return ep[np.lexsort((ep["eid"], ep["aval"]))]


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("flights", [0, 3, 100])
@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 16, 17, 32, 33, 63, 64, 65, 129])
def test_batched_equals_plain(n, flights, precision):
    from paper_2509_15377_amd import avm, workloads as W
    w = W.argon(n, band_bins=100)
    w.field = W.slab(20e-4, 120e3)  # short gap, strong field: a few electrons per primary
    w.primaries["aval"] //= 3       # up to three primaries share an avalanche
    g, f = avm.Gas(w.gas, 0), avm.Field(w.field, 0)
    out = []
    for mode, fpp in ((avm.PLAIN, 0), (avm.BATCHED, flights)):
        r = avm.Run(g, f, w.primaries, n, seed=5 + n, precision=precision, majorant=avm.BANDED, mode=mode,
                    capacity=1 << 18, flights_per_pass=fpp, band_lookahead=1.0, timeout_s=60.0)
        r.execute()
        r.sync()
        out.append((_sorted(r.endpoints()), r.counts(), r.avalanche_counts()))
        r.close()
    (a, ca, pa), (b, cb, pb) = out
    assert a.size >= n and a.tobytes() == b.tobytes()
    assert ca == cb
    assert all(np.array_equal(pa[k], pb[k]) for k in pa)


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("n,flights", [(700, 0), (9000, 0), (9000, 200), (9000, 2)])
def test_full_rings_and_long_queue(n, flights, precision):
    """Many ionisations per pass (rings overflow, the queue gets long), and a
    run whose capacity is exactly the number of its electrons."""
    from paper_2509_15377_amd import avm, workloads as W
    w = W.toy(n, band_bins=50)
    for c in w.gas.channels:
        if c.kind == W.IONISATION:
            c.values = c.values * 20.0
    w.field = W.slab(4e-4, 400e3)
    g, f = avm.Gas(w.gas, 0), avm.Field(w.field, 0)

    def go(mode, capacity, fpp):
        r = avm.Run(g, f, w.primaries, n, seed=3, precision=precision, majorant=avm.BANDED, mode=mode,
                    capacity=capacity, flights_per_pass=fpp, band_lookahead=1.0, timeout_s=60.0)
        r.execute()
        r.sync()
        out = _sorted(r.endpoints()), r.counts(), r.avalanche_counts()
        r.close()
        return out
    a, ca, pa = go(avm.PLAIN, 4 << 20, 0)
    b, cb, pb = go(avm.BATCHED, a.size, flights)
    assert a.size > 20 * n and a.tobytes() == b.tobytes()
    assert ca == cb
    assert all(np.array_equal(pa[k], pb[k]) for k in pa)
