"""Stored accumulators over rounds of workgroups: one full round and a short one after it (1089 tiles), short
lists that do not divide by the XCDs (309, 9 and 1 tiles), every tile exactly once.  A pair's accumulators
do not depend on where it sits, so every range of rows gives the same values bit for bit."""
import numpy as np
import pytest

from synth import workload as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,n_int,n_ext", [("fp16x2", 33 * 64, 33 * 64 - 5), ("fp64", 33 * 64, 33 * 32 - 3),
                                              ("fp64", 3 * 64, 103 * 32), ("fp16x2", 3 * 64, 3 * 64)])
def test_rounds(prec, n_int, n_ext):
    from paper_2507_16022_amd import dotpe
    wl = W.make_workload(9, n_int=n_int, n_ext=n_ext, n_bins=70, modes=W.MODES_HM, dets="HL", n_phi=4, snr=12.0,
                         mc_range=(10.0, 40.0), q_range=(0.3, 1.0))
    ctx = dotpe.Context(0)
    bank = ctx.load_bank(wl.h, wl.modes, wl.f, wl.ln_w_int, precision=prec)

    def lnl(**kw):
        ev = ctx.set_event(bank, d=wl.d, w=wl.w, det_r=wl.det_r, det_D=wl.det_D, ext=wl.ext, n_phi=4,
                           ln_w_ext=wl.ln_w_ext, d_max=wl.d_max, d0=wl.d0, **kw)
        out = ev.eval_lnl()["lnl"]
        ev.close()
        return out
    whole = lnl()
    assert np.all(np.isfinite(whole))
    step = max(1, n_int // 3)
    for start in range(0, n_int, step):
        count = min(step, n_int - start)
        np.testing.assert_array_equal(lnl(sub_start=start, sub_count=count), whole[start:start + count])
    np.testing.assert_array_equal(lnl(sub_start=n_int - 1, sub_count=1), whole[n_int - 1:])
    bank.close()
    ctx.close()
