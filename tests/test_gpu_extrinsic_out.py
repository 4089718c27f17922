"""Extrinsic draws come back in one copy or array by array: a draw depends on its number and the seed alone,
so calls on both sides of the limit and a call of one draw give the same leading draws."""
import numpy as np
import pytest

from synth import workload as W

pytestmark = pytest.mark.gpu


def test_extrinsic_output_paths():
    from paper_2507_16022_amd import dotpe
    wl = W.make_workload(21, n_int=40, n_ext=4, n_bins=64, modes=W.MODES_22, dets="HL", n_phi=8, snr=15.0,
                         mc_range=(10.0, 40.0), q_range=(0.3, 1.0))
    ctx = dotpe.Context(0)
    bank = ctx.load_bank(wl.h, wl.modes, wl.f, precision="fp16x2")

    def draws(n):
        return ctx.extrinsic_samples(bank, wl.d, wl.w, wl.det_r, np.full(2, -0.03), 1e-3, 64, np.array([3, 7]),
                                     np.array([0.2, -0.9]), 8, 100, 16, -0.01, 0.01, n, seed=11)
    few, most, more = draws(1), draws(32768), draws(32769)
    bank.close()
    ctx.close()
    for k in ("lat", "lon", "psi", "cos_iota", "t_geo", "ln_w"):
        assert len(more[k]) == 32769 and np.all(np.isfinite(more[k]))
        np.testing.assert_array_equal(most[k], more[k][:32768])
        assert few[k][0] == more[k][0]
    assert most["support"] == more["support"] == few["support"]
    assert few["n_eff_prior"] == pytest.approx(1.0)
