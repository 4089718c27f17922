"""Events between the fused kernel's fast pass and the bound pass with listed survivors: from 256 tiles
of 128 x 128 on, the bound pass leaves every tile with a survivor to the coefficient route.  Around the
limits (255, 256 and 260 tiles, ragged edges, three chunks of tiles), loud and quiet, against the fast
pass: the same pairs evaluated from the same accumulators, so the same sums and top-k (1e-12: sums over
tiles in one order), the same counts, and the certificate on both sides."""
import numpy as np
import pytest

from synth import workload as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_int,n_ext,prec,snr", [
    (255 * 128, 128, "fp16x2", 20.0), (2047, 2047, "fp16x2", 12.0), (2048, 2048, "bf16x2", 20.0),
    (2560, 3329, "fp16x2", 20.0), (16385, 1030, "fp16x2", 9.5), (16385, 1030, "fp16x2", 25.0)])
def test_mid_events(n_int, n_ext, prec, snr):
    from paper_2507_16022_amd import dotpe
    wl = W.make_workload(3, n_int=n_int, n_ext=n_ext, n_bins=48, modes=W.MODES_HM, dets="HL", n_phi=16,
                         snr=snr, mc_range=(10.0, 40.0), q_range=(0.3, 1.0))
    ctx = dotpe.Context(0)
    bank = ctx.load_bank(wl.h, wl.modes, wl.f, wl.ln_w_int, precision=prec)
    res = []
    for flags in (0, dotpe.FLAG_NO_BOUND_PASS):
        ev = ctx.set_event(bank, d=wl.d, w=wl.w, det_r=wl.det_r, det_D=wl.det_D, ext=wl.ext, n_phi=16,
                           ln_w_ext=wl.ln_w_ext, d_max=wl.d_max, d0=wl.d0, n_norm=wl.n_norm,
                           cut_delta=30.0, top_k=32, topk_window=12.0, flags=flags)
        res.append(ev.evidence())
        ev.close()
    bank.close()
    ctx.close()
    a, b = res
    print(f"{n_int} x {n_ext} {prec}: rerun {a['n_tiles_rerun']} / {b['n_tiles_rerun']}, cut "
          f"{a['cut_delta_used']}, passes {a['n_passes']} / {b['n_passes']}, triples {a['n_triples_marg']}",
          flush=True)
    assert a["n_tiles_listed"] == 0 and a["n_tiles_rerun"] >= b["n_tiles_rerun"]
    for k in ("n_pairs", "n_pairs_bounded", "n_triples_marg", "n_passes", "topk_count"):
        assert a[k] == b[k], k
    for k in ("ln_z", "ln_sum_p", "ln_sum_p2", "ln_sum_row2", "ln_sum_col2", "max_ln_p", "max_lnl_ml"):
        assert a[k] == pytest.approx(b[k], rel=1e-12), k
    assert a["ln_z"] <= a["ln_z_upper"] + 1e-12 and a["ln_z_upper"] >= b["ln_z_upper"] - 1e-9
    for k in ("topk_i", "topk_e", "topk_o"):
        np.testing.assert_array_equal(a[k], b[k])
    np.testing.assert_allclose(a["topk_lnp"], b["topk_lnp"], rtol=1e-13)
