"""ln L of tiles of few pairs, FP64 bank: the sum over the phases in FP64, so that values near zero (a weak
signal, a far prior) are as close to the plain sum over the phases as the distance rule's values are."""
import numpy as np
import pytest

from oracle import oracle as O
from synth import workload as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_int,n_ext,n_phi", [(1, 1, 32), (5, 3, 4), (3, 40, 128), (65, 1, 17), (1, 33, 7)])
def test_few_pairs(n_int, n_ext, n_phi):
    from paper_2507_16022_amd import dotpe
    wl = W.make_workload(4, n_int=n_int, n_ext=n_ext, n_bins=64, modes=W.MODES_HM, dets="HL", n_phi=n_phi, snr=1.0,
                         mc_range=(10.0, 40.0), q_range=(0.3, 1.0))
    ctx = dotpe.Context(0)
    bank = ctx.load_bank(wl.h, wl.modes, wl.f, None, precision="fp64")
    ev = ctx.set_event(bank, d=wl.d, w=wl.w, det_r=wl.det_r, det_D=wl.det_D, ext=wl.ext, n_phi=n_phi, d_max=1e6,
                       d0=1.0)
    got = ev.eval_lnl(triples=True)
    ev.close()
    z = (got["dh"] / np.sqrt(got["hh"])).ravel()
    v = ctx.distmarg(got["dh"].ravel(), got["hh"].ravel(), 1.0 / 1e6).reshape(got["dh"].shape)
    bank.close()
    ctx.close()
    assert np.all(np.isfinite(z))
    m = v.max(-1)
    ref = m + np.log(np.mean(np.exp(v - m[..., None]), -1))
    # the library's own values per phase, summed here: rounding of up to 128 terms
    assert np.max(np.abs(got["lnl"] - ref)) <= 1e-12 * (1 + np.max(np.abs(ref)))
    # and the plain rule: its table's 1e-7
    assert np.max(np.abs(v - O.ln_dist_marg(got["dh"], got["hh"], 1e6, 1.0))) <= 2e-7
