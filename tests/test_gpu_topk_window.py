"""Top-k through the window: few candidates within it (counted places), some hundreds (the network in
LDS), more than fit (the whole network), all equal to a sort of the ln p of every pair."""
import numpy as np
import pytest

from synth import workload as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("window,k", [(0.5, 16), (2.0, 300), (4.0, 1000), (9.0, 64), (13.0, 300), (17.0, 4096), (25.0, 4096), (60.0, 700)])
def test_topk_window(window, k):
    from paper_2507_16022_amd import dotpe
    wl = W.make_workload(4, n_int=130, n_ext=140, n_bins=48, modes=W.MODES_HM, dets="HL", n_phi=8, snr=9.0,
                         mc_range=(10.0, 40.0), q_range=(0.3, 1.0), random_weights=True)
    ctx = dotpe.Context(0)
    bank = ctx.load_bank(wl.h, wl.modes, wl.f, wl.ln_w_int, precision="fp64")
    ev = ctx.set_event(bank, d=wl.d, w=wl.w, det_r=wl.det_r, det_D=wl.det_D, ext=wl.ext, n_phi=8,
                       ln_w_ext=wl.ln_w_ext, d_max=wl.d_max, d0=wl.d0, top_k=k, topk_window=window)
    lnp = ev.eval_lnl()["lnl"] + wl.ln_w_int[:, None] + wl.ln_w_ext[None, :]
    r = ev.evidence()
    ev.close()
    bank.close()
    ctx.close()
    flat = lnp.ravel()
    order = np.argsort(-flat, kind="stable")[:k]
    order = order[flat[order] >= flat.max() - window]
    within = int(np.sum(flat >= flat.max() - window))
    print(f"window {window}: {within} pairs within it, {r['topk_count']} reported", flush=True)
    assert r["topk_exact"] == 1 and r["topk_count"] == len(order)
    np.testing.assert_allclose(r["topk_lnp"], flat[order], rtol=1e-12)
    np.testing.assert_array_equal(r["topk_i"] * lnp.shape[1] + r["topk_e"], order)
