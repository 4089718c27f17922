"""Evidence over 79 to 128 phases and more than 512 tiles: shorter turns of the marginalisation, so that three
workgroups share a CU; equal to the sums over the ln L matrix of the same event, whose turns are the longer ones."""
import numpy as np
import pytest

from synth import workload as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,modes,n_phi,snr,cut", [
    ("fp16x2", W.MODES_HM, 79, 8.0, 0.0), ("fp16x2", W.MODES_HM, 128, 14.0, 40.0),
    ("bf16x2", ((2, 2), (2, 1), (3, 3)), 100, 8.0, 0.0), ("fp16x2", W.MODES_HM, 78, 8.0, 0.0)])
def test_many_phases(prec, modes, n_phi, snr, cut):
    from paper_2507_16022_amd import dotpe
    n_int, n_ext = 27 * 64 - 3, 20 * 64 - 5                # 540 tiles
    wl = W.make_workload(12, n_int=n_int, n_ext=n_ext, n_bins=40, modes=modes, dets="HL", n_phi=n_phi, snr=snr,
                         mc_range=(10.0, 40.0), q_range=(0.3, 1.0), random_weights=True)
    ctx = dotpe.Context(0)
    bank = ctx.load_bank(wl.h, wl.modes, wl.f, wl.ln_w_int, precision=prec)
    ev = ctx.set_event(bank, d=wl.d, w=wl.w, det_r=wl.det_r, det_D=wl.det_D, ext=wl.ext, n_phi=n_phi,
                       ln_w_ext=wl.ln_w_ext, d_max=wl.d_max, d0=wl.d0, cut_delta=cut)
    lnp = ev.eval_lnl()["lnl"] + wl.ln_w_int[:, None] + wl.ln_w_ext[None, :]
    r = ev.evidence()
    ev.close()
    bank.close()
    ctx.close()
    m = lnp.max()
    ref = m + np.log(np.sum(np.exp(lnp - m)))
    # the same values per pair, summed in another order; cut triples lie 40 below
    assert abs(r["ln_sum_p"] - ref) <= 1e-9 * (1 + abs(ref))
    assert r["max_ln_p"] == pytest.approx(m, rel=1e-9)
    rows = np.exp(lnp - m).sum(1)
    assert r["ln_sum_row2"] - 2 * m == pytest.approx(np.log(np.sum(rows ** 2)), abs=1e-8)
