"""The ring of waiting electrons in each wave: with the induced signal on, and
when the time budget ends while electrons wait there."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _many_ionisations(n):
    """Several ionisations per pass in every wave: rings overflow, the queue gets long."""
    from paper_2509_15377_amd import workloads as W
    w = W.toy(n, band_bins=50)
    for c in w.gas.channels:
        if c.kind == W.IONISATION:
            c.values = c.values * 20.0
    w.field = W.slab(4e-4, 400e3)
    return w


def test_signal_through_full_rings(oracle_mod):
    """Bin by bin against the oracle, for the avalanches all of whose electrons
    took the oracle's decisions (deposits are atomics: the bar is that of the
    other signal tests, 1e-9 of the row's largest bin)."""
    from oracle import compare
    from paper_2509_15377_amd import avm
    n, spec = 9000, (0.0, 2e-4, 60)
    w = _many_ionisations(n)
    ref, sig = oracle_mod.run(oracle_mod.Gas(w.gas), w.field, w.primaries, 3, banded=True, band_lookahead=1.0,
                              signal=spec + (n,))
    ep, _, _, got = avm.run(w, seed=3, majorant=avm.BANDED, band_lookahead=1.0, capacity=1 << 20, signal=spec,
                            timeout_s=60.0)
    compare.assert_parity(ep, ref)
    assert ref.size > 20 * n
    pairs = [set(zip(a["aval"].tolist(), a["eid"].tolist(), a["trace"].tolist(), a["n_null"].tolist()))
             for a in (ep, ref)]
    flipped = np.array(sorted({aval for aval, *_ in pairs[0] ^ pairs[1]}), dtype=np.int64)
    same = np.setdiff1d(np.arange(n), flipped)
    print("avalanches with other decisions:", flipped.size)
    assert same.size > 0.9 * n
    scale = np.maximum(np.abs(sig).max(axis=1, keepdims=True), 1e-12)
    assert (np.abs(got - sig) / scale)[same].max() <= 1e-9


def test_time_budget_ends_with_electrons_waiting():
    """Every electron that was created has its start record, and the next call
    (the same scratch memory) is not touched by what was left."""
    import torch

    from paper_2509_15377_amd import avm, workloads as W
    w = W.batched(1024, band_bins=100)
    g, f = avm.Gas(w.gas, 0), avm.Field(w.field, 0)
    prim = torch.from_numpy(w.primaries.view(np.uint8).copy()).to("cuda:0")
    stream = torch.cuda.current_stream()
    kw = dict(seed=w.seed, majorant=avm.BANDED, band_lookahead=1.0, stream=stream)
    cap = avm.NOALLOC_MAX_ELECTRONS
    out = avm.noalloc_outputs(cap, w.n_aval)
    for k in ("x0", "y0", "z0", "t0", "e0"):
        out[k].fill_(float("nan"))
    out["eid"].zero_()
    out["avalanche"].fill_(-1)
    print("time budget of 12 ms", flush=True)
    avm.run_noalloc(g, f, prim, w.n_aval, out, timeout_s=12e-3, **kw)
    stream.synchronize()
    _, tot, _, flags = avm.noalloc_results(out, w.n_aval)
    assert flags & avm.NOALLOC_TIMEOUT
    n = min(tot["n_requested"], cap)
    print(n, "electrons,", n - tot["n_endpoints"], "of them alive", flush=True)
    assert n - tot["n_endpoints"] > 16 * w.n_aval
    for k in ("x0", "y0", "z0", "t0", "e0"):
        assert bool(torch.isfinite(out[k][:n]).all()), k
    assert bool((out["eid"][:n] != 0).all())
    aval = out["avalanche"][:n]
    assert bool(((aval >= 0) & (aval < w.n_aval)).all())

    small = W.argon(40, band_bins=100)
    g, f = avm.Gas(small.gas, 0), avm.Field(small.field, 0)
    prim = torch.from_numpy(small.primaries.view(np.uint8).copy()).to("cuda:0")
    kw["seed"] = small.seed
    out = avm.noalloc_outputs(1 << 18, small.n_aval)
    avm.run_noalloc(g, f, prim, small.n_aval, out, timeout_s=30.0, **kw)
    stream.synchronize()
    ep, tot, _, flags = avm.noalloc_results(out, small.n_aval)
    ref, rtot, _ = avm.run(small, capacity=1 << 18, majorant=avm.BANDED, band_lookahead=1.0, timeout_s=30.0)
    assert flags == 0 and tot["n_real"] == rtot["n_real"]
    key = lambda a: a[np.lexsort((a["eid"], a["aval"]))].tobytes()
    assert key(ep) == key(ref)
