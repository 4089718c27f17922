"""The bound pass over more workgroups than one dimension of a grid may number (2^23 bank rows x 2^14 samples:
2^24 workgroups, 2^32 work-items), and over several rows of the grid with a last one that is not full: the
event gives the sums and the best pair of its halves."""
import numpy as np
import pytest

from synth import workload as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_int,n_ext", [(1 << 20, 8192 + 65), (1 << 23, 1 << 14)])
def test_bound_grid(n_int, n_ext):
    import torch
    from paper_2507_16022_amd import dotpe
    wl = W.make_workload(8, n_int=n_int, n_ext=n_ext, n_bins=64, modes=W.MODES_22, dets="HL", n_phi=4, snr=20.0,
                         mc_range=(10.0, 40.0), q_range=(0.3, 1.0), with_bank=False)
    h = W.bank_on_device(torch, wl.meta["mc"], wl.meta["q"], wl.meta["chi"], wl.f, wl.modes, chunk=1 << 18)
    ctx = dotpe.Context(0)
    bank = ctx.load_bank(h, wl.modes, wl.f, precision="fp16x2")
    del h
    torch.cuda.empty_cache()

    def evidence(start, count):
        ev = ctx.set_event(bank, d=wl.d, w=wl.w, det_r=wl.det_r, det_D=wl.det_D, ext=wl.ext, n_phi=4,
                           d_max=wl.d_max, d0=wl.d0, cut_delta=30.0, top_k=4, topk_window=5.0, sub_start=start,
                           sub_count=count)
        r = ev.evidence()
        ev.close()
        print(f"{count} x {n_ext}: {r['t_fused_ms']:.1f} ms, bounded {r['n_pairs_bounded']} of {r['n_pairs']}",
              flush=True)
        return r
    half = n_int // 2
    whole, a, b = evidence(0, n_int), evidence(0, half), evidence(half, n_int - half)
    bank.close()
    ctx.close()
    assert whole["n_pairs"] == n_int * n_ext and whole["n_pairs_bounded"] > 0.9 * whole["n_pairs"]
    # the halves cut at their own maxima, 30 below: what they evaluate beyond the whole is below e^-30 a pair
    assert whole["ln_sum_p"] == pytest.approx(np.logaddexp(a["ln_sum_p"], b["ln_sum_p"]), abs=1e-6)
    best = max((a, b), key=lambda r: r["max_ln_p"])
    assert whole["max_ln_p"] == best["max_ln_p"]
    assert whole["topk_i"][0] == best["topk_i"][0] and whole["topk_e"][0] == best["topk_e"][0]
