"""Stored accumulators of split banks: a list of more than 512 tiles is taken a tile per workgroup, a
shorter one in halves of 32 rows.  A pair's accumulators do not depend on where it sits, so the ln L
matrix of a whole event (529 to 640 tiles, a last band of 1 to 7 tile rows, ragged edges) equals, bit for
bit, that of ranges of its rows (2 to 36 tiles) and of scattered rows; one and four m groups."""
import numpy as np
import pytest

from synth import workload as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,modes,n_int,n_ext", [("fp16x2", "hm", 23 * 64, 23 * 64), ("bf16x2", "hm", 1473, 1601),
                                                    ("fp16x2", "22", 40 * 64 - 1, 16 * 64 - 33)])
def test_tiles_and_halves(prec, modes, n_int, n_ext):
    from paper_2507_16022_amd import dotpe
    wl = W.make_workload(9, n_int=n_int, n_ext=n_ext, n_bins=70, modes=W.MODES_22 if modes == "22" else W.MODES_HM,
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
    for start, count in ((0, 1), (5, 64), (n_int - 65, 65), (n_int - 33, 33)):
        np.testing.assert_array_equal(lnl(sub_start=start, sub_count=count), whole[start:start + count])
    idx = np.random.default_rng(1).permutation(n_int)[:77].astype(np.int64)
    np.testing.assert_array_equal(lnl(sub_idx=idx), whole[idx])
    bank.close()
    ctx.close()
