"""Kept phases in turns of the distance rule: fewer per turn below 64 phases with FP64 accumulators.  Phase
counts on both sides, blocks of phases that do not divide a turn, one to 128 phases, every pair kept and cut,
against the materialised matrix of the same event and the oracle's ln L."""
import numpy as np
import pytest

from oracle import oracle as O
from synth import workload as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp64", "fp16x2"])
@pytest.mark.parametrize("n_phi", [1, 17, 63, 64, 65, 128])
def test_turns(prec, n_phi):
    from paper_2507_16022_amd import dotpe
    wl = W.make_workload(4, n_int=131, n_ext=97, n_bins=64, modes=W.MODES_HM, dets="HL", n_phi=n_phi, snr=8.0,
                         mc_range=(10.0, 40.0), q_range=(0.3, 1.0))
    ctx = dotpe.Context(0)
    bank = ctx.load_bank(wl.h, wl.modes, wl.f, wl.ln_w_int, precision=prec)
    ev = ctx.set_event(bank, d=wl.d, w=wl.w, det_r=wl.det_r, det_D=wl.det_D, ext=wl.ext, n_phi=n_phi,
                       ln_w_ext=wl.ln_w_ext, d_max=wl.d_max, d0=wl.d0, cut_delta=0.0)
    r = ev.evidence()
    lnl = ev.eval_lnl()["lnl"]
    ev.close()
    bank.close()
    ctx.close()
    assert r["n_triples_marg"] == lnl.size * n_phi
    m = lnl.max()
    # the same values summed in another order
    assert r["ln_sum_p"] == pytest.approx(m + np.log(np.sum(np.exp(lnl - m))), abs=1e-10)
    rows, cols = [0, 64, 130], [0, 63, 96]
    ref = O.eval_lnl(wl.subset(rows, cols))["lnl"]
    # the distance rule's table (1e-6); FP16x2 operands besides (1e-6 of lnL^ML, tens here)
    np.testing.assert_allclose(lnl[np.ix_(rows, cols)], ref, rtol=0, atol=1e-6 if prec == "fp64" else 1e-3)
