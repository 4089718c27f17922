"""The pre-selection's kernels off the usual shapes: six to eight channels (one detector per pass of the
Gram sums), more detectors than a pass of five channels takes, one to three waves per workgroup, phase
grids whose forms leave room for one workgroup per CU; bank rows shared through LDS and not."""
import numpy as np
import pytest

from oracle import oracle as O
from synth import workload as W

pytestmark = pytest.mark.gpu

MODES8 = ((2, 2), (2, 1), (3, 3), (3, 2), (4, 4), (3, 1), (4, 3), (4, 2))


@pytest.mark.parametrize("nc,n_det,n_bins,n_t,n_phi", [
    (1, 2, 70, 32, 128), (2, 3, 50, 96, 48), (3, 1, 64, 96, 128), (5, 4, 100, 128, 32), (5, 2, 33, 64, 64),
    (6, 2, 65, 32, 24), (6, 3, 128, 128, 32), (7, 2, 90, 64, 128), (8, 2, 40, 32, 32), (8, 3, 70, 96, 128),
    (8, 8, 33, 64, 16)])
def test_preselect_shapes(nc, n_det, n_bins, n_t, n_phi):
    from paper_2507_16022_amd import dotpe
    rng = np.random.default_rng(nc * 100 + n_t)
    n, modes = 45, MODES8[:nc]
    f = np.geomspace(20.0, 512.0, n_bins)
    h = rng.normal(size=(n, nc, n_bins)) + 1j * rng.normal(size=(n, nc, n_bins))
    d = rng.normal(size=(n_det, n_bins)) + 1j * rng.normal(size=(n_det, n_bins))
    w = rng.uniform(0.5, 2.0, (n_det, n_bins))
    ci = rng.uniform(-1.0, 1.0, n)
    t0, dt = rng.uniform(-0.1, 0.0, n_det), 1e-3
    ctx = dotpe.Context(0)
    bank = ctx.load_bank(h, modes, f, precision="fp16x2")
    r = ctx.preselect(bank, d, w, t0, dt, n_t, ci, n_phi)
    bank.close()
    ctx.close()
    rows = np.array([0, 17, 31, 32, n - 1])
    _, per = O.incoherent_ml(h[rows], modes, ci[rows], f, d, w, t0, dt, n_t, n_phi)
    # FP16x2 operands and FP32 accumulation: ~1e-6 relative in each projection
    assert np.all(np.abs(r["lnl_det"][rows] - per) <= 1e-3 + 4e-6 * np.abs(per))
