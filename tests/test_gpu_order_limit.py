"""The coefficient route's list put in order at the most tiles its bitmap holds (2^19 tiles, 64 KB of LDS
besides the kernel's own sums), and one tile row more, where the list stays as it is: an event gives the sums
and the best pairs of its two halves."""
import numpy as np
import pytest

from synth import workload as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_int,n_ext", [(1 << 20, 2048), (1 << 17, 16384), ((1 << 17) + 64, 16384)])
def test_order_at_the_most_tiles(n_int, n_ext):
    import torch
    from paper_2507_16022_amd import dotpe
    wl = W.make_workload(6, n_int=n_int, n_ext=n_ext, n_bins=64, modes=W.MODES_22, dets="HL", n_phi=8, snr=14.0,
                         mc_range=(10.0, 40.0), q_range=(0.3, 1.0), with_bank=False)
    h = W.bank_on_device(torch, wl.meta["mc"], wl.meta["q"], wl.meta["chi"], wl.f, wl.modes)
    ctx = dotpe.Context(0)
    bank = ctx.load_bank(h, wl.modes, wl.f, precision="fp16x2")
    del h
    torch.cuda.empty_cache()

    def evidence(start, count):
        ev = ctx.set_event(bank, d=wl.d, w=wl.w, det_r=wl.det_r, det_D=wl.det_D, ext=wl.ext, n_phi=8,
                           d_max=wl.d_max, d0=wl.d0, cut_delta=40.0, top_k=8, topk_window=10.0, sub_start=start,
                           sub_count=count)
        r = ev.evidence()
        ev.close()
        return r
    half = n_int // 2
    whole, a, b = evidence(0, n_int), evidence(0, half), evidence(half, n_int - half)
    bank.close()
    ctx.close()
    assert whole["n_tiles_rerun"] >= 1024, whole["n_tiles_rerun"]
    assert whole["n_pairs"] == n_int * n_ext
    # the halves cut at their own maxima, 40 below: what one of them evaluates beyond the other is below e^-40
    # of its sum per pair
    assert whole["ln_sum_p"] == pytest.approx(np.logaddexp(a["ln_sum_p"], b["ln_sum_p"]), abs=1e-6)
    assert whole["max_ln_p"] == max(a["max_ln_p"], b["max_ln_p"])
    best = max((a, b), key=lambda r: r["max_ln_p"])
    assert whole["topk_i"][0] == best["topk_i"][0] and whole["topk_e"][0] == best["topk_e"][0]
