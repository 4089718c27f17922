"""The pre-selection's phase maximum for every kind of phase grid: powers of two (phases that share
their products by symmetry, from the smallest grid with four) and other counts; one, two and five
channels of odd and even m; row blocks that end inside a 32-row block for one to three detectors."""
import numpy as np
import pytest

from oracle import oracle as O
from synth import workload as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("modes,dets", [(W.MODES_22, "H"), (((2, 1), (3, 3)), "HL"), (W.MODES_HM, "HLV")])
@pytest.mark.parametrize("n_phi", [1, 2, 3, 4, 8, 12, 32, 128])
def test_preselect_phase_grids(modes, dets, n_phi):
    from paper_2507_16022_amd import dotpe
    n = 45
    wl = W.make_workload(31, n_int=n, n_ext=4, n_bins=64, modes=modes, dets=dets, n_phi=n_phi, snr=15.0,
                         mc_range=(8.0, 40.0), q_range=(0.2, 0.9), chi_range=(-0.5, 0.5))
    ci = np.random.default_rng(n_phi).uniform(-1.0, 1.0, n)
    n_t, dt = 32, 1e-3
    t0 = np.full(len(dets), -0.5 * n_t * dt)
    ctx = dotpe.Context(0)
    bank = ctx.load_bank(wl.h, wl.modes, wl.f, precision="fp16x2")
    r = ctx.preselect(bank, wl.d, wl.w, t0, dt, n_t, ci, n_phi)
    bank.close()
    ctx.close()
    rows = np.arange(0, n, 11)           # the first and last row of blocks among them
    rows = np.unique(np.concatenate([rows, [31, 32, n - 1]]))
    _, per = O.incoherent_ml(wl.h[rows], wl.modes, ci[rows], wl.f, wl.d, wl.w, t0, dt, n_t, n_phi)
    # FP16x2 operands and FP32 accumulation: ~1e-6 relative in each projection
    assert np.all(np.abs(r["lnl_det"][rows] - per) <= 1e-3 + 4e-6 * np.abs(per))
