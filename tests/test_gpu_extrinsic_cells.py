"""Extrinsic draws at the edges of the cell blocks and row blocks: one cell, fewer cells than a
block of 256, blocks that end inside a sky point's times, one row, more rows than a 32-row block,
the largest number of rows; a component whose cells all lie off the grids."""
import numpy as np
import pytest

from oracle import oracle as O
from synth import workload as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("C,S,J,n_s", [(1, 1, 1, 3), (33, 7, 50, 400), (64, 40, 13, 1000), (3, 300, 61, 5)])
def test_extrinsic_cells(C, S, J, n_s):
    from paper_2507_16022_amd import dotpe
    wl = W.config_tiny(seed=12, n_int=96, n_ext=4, snr=18.0)
    rng = np.random.default_rng(C)
    rows = rng.permutation(96)[:C]
    ci = rng.uniform(-1, 1, C)
    n_t, dt, n_phi, seed = 64, 1e-3, 4, 9
    t0 = np.full(2, -0.5 * n_t * dt)
    lo, hi = -0.01, 0.01
    ctx = dotpe.Context(0)
    bank = ctx.load_bank(wl.h, wl.modes, wl.f, wl.ln_w_int)
    g = ctx.extrinsic_samples(bank, wl.d, wl.w, wl.det_r, t0, dt, n_t, rows, ci, n_phi, S, J, lo, hi,
                              n_s, seed=seed)
    off = ctx.extrinsic_samples(bank, wl.d, wl.w, wl.det_r, t0 + 1e3, dt, n_t, rows, ci, n_phi, S, J,
                                lo, hi, n_s, seed=seed)
    bank.close()
    ctx.close()
    rho2 = O.arrival_time_series(wl.h[rows], wl.modes, ci, wl.f, wl.d, wl.w, t0, dt, n_t, n_phi)
    lat, lon = O.fibonacci_sky(S)
    lnW, lnZ = O.proposal_table(rho2, t0, dt, wl.det_r, lat, lon, lo, hi, J, 0.5)
    ref = O.extrinsic_proposal(lnW, lnZ, lat, lon, lo, hi, n_s, seed)
    same = (np.abs(g["lat"] - ref["lat"]) < 1e-9) & (np.abs(g["t_geo"] - ref["t_geo"]) < 1e-12)
    # the series carry FP32 rounding (rho^2 ~ 300: 1e-4), so a draw near a cell's edge may move
    assert same.mean() >= 0.97
    assert np.max(np.abs(g["ln_w"][same] - ref["ln_w"][same])) < 1e-2
    assert np.allclose(g["psi"], ref["psi"], rtol=1e-14, atol=0)
    assert g["support"] == pytest.approx(np.mean(np.exp(lnW - lnZ[:, None, None]).mean(0) > 0), abs=1e-2)
    # every cell off the grids: no support, the draws stay inside the cells
    assert off["support"] == 0.0 and np.all(np.isin(np.round(off["lat"], 9), np.round(lat, 9)))
