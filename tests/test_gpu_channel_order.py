"""Gases whose channel 0 is not an elastic channel without a window (the
flight step takes that one without reading its parameters): per trajectory
against the oracle, and batched against plain in both precisions."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _gas(kind):
    from paper_2509_15377_amd import workloads as W
    g = W.argon_like_gas(band_bins=100)
    if kind == "reversed":
        g.channels = g.channels[::-1]
    elif kind == "excitation first":
        g.channels = g.channels[1:] + g.channels[:1]
    elif kind == "elastic window":
        g.channels[0].e_lo_eV = 0.4
        g.channels[0].e_hi_eV = 30.0
    return g


@pytest.mark.parametrize("kind", ["reversed", "excitation first", "elastic window"])
def test_channel_order(kind):
    from oracle import compare, oracle as O
    from paper_2509_15377_amd import avm, workloads as W
    w = W.argon(12)
    w.field = W.slab(60e-4, 45e3)
    gas = _gas(kind)
    g, f = avm.Gas(gas, 0), avm.Field(w.field, 0)

    def go(mode, precision):
        r = avm.Run(g, f, w.primaries, w.n_aval, seed=9, precision=precision, majorant=avm.BANDED, mode=mode,
                    capacity=1 << 19, band_lookahead=1.0, timeout_s=60.0)
        r.execute()
        r.sync()
        ep = r.endpoints()
        r.close()
        return ep[np.lexsort((ep["eid"], ep["aval"]))]
    ep = go(avm.BATCHED, avm.FP64)
    ref = O.run(O.Gas(gas), w.field, w.primaries, 9, banded=True, band_lookahead=1.0)
    compare.assert_parity(ep, ref)
    assert ep["n_masked"].sum() > 0 or kind != "elastic window"
    assert ep.tobytes() == go(avm.PLAIN, avm.FP64).tobytes()
    assert go(avm.BATCHED, avm.FP32_MIXED).tobytes() == go(avm.PLAIN, avm.FP32_MIXED).tobytes()
