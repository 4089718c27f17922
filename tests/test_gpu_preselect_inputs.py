"""Pre-selection with host inputs of all lengths: data (and weights) long enough to be copied from where they are
between small ones that are copied as one piece; row inputs short and long."""
import numpy as np
import pytest

from oracle import oracle as O

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,n_det,n_bins", [(5, 8, 1100), (20, 5, 900), (9000, 1, 40), (8500, 8, 600)])
def test_inputs(n, n_det, n_bins):
    from paper_2507_16022_amd import dotpe
    rng = np.random.default_rng(n)
    f = np.geomspace(20.0, 512.0, n_bins)
    h = rng.normal(size=(n, 1, n_bins)) + 1j * rng.normal(size=(n, 1, n_bins))
    d = rng.normal(size=(n_det, n_bins)) + 1j * rng.normal(size=(n_det, n_bins))
    w = rng.uniform(0.5, 2.0, (n_det, n_bins))
    ci = rng.uniform(-1.0, 1.0, n)
    t0, dt = rng.uniform(-0.1, 0.0, n_det), 1e-3
    ctx = dotpe.Context(0)
    bank = ctx.load_bank(h, ((2, 2),), f, precision="fp16x2")
    r = ctx.preselect(bank, d, w, t0, dt, 32, ci, 8)
    bank.close()
    ctx.close()
    rows = np.array([0, 1, n - 1])
    _, per = O.incoherent_ml(h[rows], ((2, 2),), ci[rows], f, d, w, t0, dt, 32, 8)
    # FP16x2 operands and FP32 accumulation: ~1e-6 relative in each projection
    assert np.all(np.abs(r["lnl_det"][rows] - per) <= 1e-3 + 4e-6 * np.abs(per))
