"""Stored accumulators of few tiles: halves by two waves (up to 128 tiles), tiles by four waves (up to 512), both
with more stages than an event of one mode and few bins has chunks, against the kernel of more tiles.  A pair's
accumulators do not depend on the kernel, so ranges of rows give the whole event's ln L bit for bit."""
import numpy as np
import pytest

from synth import workload as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,modes,n_bins", [("fp16x2", "22", 17), ("fp16x2", "hm", 150), ("bf16x2", "hm", 60),
                                               ("bf16x2", "22", 300)])
def test_few_tiles(prec, modes, n_bins):
    from paper_2507_16022_amd import dotpe
    n_int, n_ext = 33 * 64, 16 * 64 - 5                # 528 tiles
    wl = W.make_workload(9, n_int=n_int, n_ext=n_ext, n_bins=n_bins, modes=W.MODES_22 if modes == "22" else W.MODES_HM,
                         dets="HL", n_phi=4, snr=12.0, mc_range=(10.0, 40.0), q_range=(0.3, 1.0))
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
    # 16 to 512 tiles: 1, 8, 9, 16, 17 and 32 rows of tiles, the last ones ragged
    for start, count in ((64, 64), (0, 8 * 64), (n_int - 9 * 64, 9 * 64), (3, 16 * 64), (64, 16 * 64 + 63), (64, 32 * 64)):
        np.testing.assert_array_equal(lnl(sub_start=start, sub_count=count), whole[start:start + count])
    bank.close()
    ctx.close()
