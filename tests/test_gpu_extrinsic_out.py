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


def test_extrinsic_most_draws():
    """More draws than a grid of one dimension has waves for (2^26): the first ones are those of a short call,
    the last ones carry their own numbers' uniforms."""
    from oracle import oracle as O
    from paper_2507_16022_amd import dotpe
    wl = W.make_workload(21, n_int=40, n_ext=4, n_bins=64, modes=W.MODES_22, dets="HL", n_phi=8, snr=15.0,
                         mc_range=(10.0, 40.0), q_range=(0.3, 1.0))
    ctx = dotpe.Context(0)
    bank = ctx.load_bank(wl.h, wl.modes, wl.f, precision="fp16x2")
    n = (1 << 26) + 5

    def draws(n):
        return ctx.extrinsic_samples(bank, wl.d, wl.w, wl.det_r, np.full(2, -0.03), 1e-3, 64, np.array([3, 7]),
                                     np.array([0.2, -0.9]), 8, 20, 5, -0.01, 0.01, n, seed=11)
    few, all_ = draws(1000), draws(n)
    bank.close()
    ctx.close()
    for k in ("lat", "lon", "psi", "cos_iota", "t_geo", "ln_w"):
        assert len(all_[k]) == n
        np.testing.assert_array_equal(all_[k][:1000], few[k])
    q = np.arange(n - 100, n, dtype=np.uint64)
    u = np.array([O.splitmix64_uniform(11, int(4 * x + 3)) for x in q])
    np.testing.assert_allclose(all_["cos_iota"][-100:], 2.0 * u - 1.0, rtol=0, atol=1e-15)
    assert np.all(np.isin(all_["lat"][-100:], np.unique(few["lat"]))) and np.all(np.isfinite(all_["ln_w"][-100:]))
