"""Electrons at rest in a zero field, in gases with a rate at zero energy:
every collision's outcome in both precisions and modes is the oracle's, with
one channel and with a second one whose window is shut."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

KMAX = 500


def _gas(channels):
    from paper_2509_15377_amd import workloads as W
    g = W.constant_rate_gas(40.0, mass_ratio=1.37e-5)
    g.band_bins = 10
    if channels == 2:
        g.channels.append(W.Channel(W.EXCITATION, np.full(g.n_bins + 1, 25.0), values_kind=W.VALUES_RATE,
                                    loss_eV=11.5, e_lo_eV=11.5))
    return g


@pytest.mark.parametrize("majorant", ["global", "banded"])
@pytest.mark.parametrize("channels", [1, 2])
def test_at_rest(channels, majorant):
    from oracle import oracle as O
    from paper_2509_15377_amd import avm, workloads as W
    gas, field = _gas(channels), W.slab(1.0, 0.0)
    prim = W.primaries_at_rest(70, z=0.5)
    banded = majorant == "banded"
    ref = O.run(O.Gas(gas), field, prim, 21, banded=banded, k_max=KMAX, band_lookahead=1.0 if banded else 0.0)
    assert ref["n_real"].sum() > 15000 and (channels == 1 or ref["n_masked"].sum() > 10000)
    g, f = avm.Gas(gas, 0), avm.Field(field, 0)
    for mode in (avm.BATCHED, avm.PLAIN):
        for precision in (avm.FP64, avm.FP32_MIXED):
            print(channels, majorant, mode, precision, flush=True)
            r = avm.Run(g, f, prim, prim.size, seed=21, mode=mode, precision=precision, k_max=KMAX, capacity=1024,
                        majorant=avm.BANDED if banded else avm.GLOBAL, band_lookahead=1.0 if banded else 0.0,
                        timeout_s=30.0)
            r.execute()
            r.sync()
            ep = r.endpoints()
            r.close()
            ep = ep[np.lexsort((ep["eid"], ep["aval"]))]
            for k in ("eid", "status", "n_real", "n_ion", "n_null", "n_masked", "n_band", "trace"):
                assert np.array_equal(ep[k], ref[k]), (mode, precision, k)
            assert (ep["e1"] == 0.0).all() and (ep["z1"] == 0.5).all()
