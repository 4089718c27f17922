"""The row-side (h|h) operand of split banks, through the (h|h) of every triple: one to eight channels,
bins that do not fill a lane's turn or a chunk, one to four detectors (more than one pass of
accumulators), row counts around the 16 rows of a workgroup, scattered rows."""
import numpy as np
import pytest

from oracle import oracle as O
from synth import workload as W

pytestmark = pytest.mark.gpu

MODES8 = ((2, 2), (2, 1), (3, 3), (3, 2), (4, 4), (3, 1), (4, 3), (4, 2))


@pytest.mark.parametrize("prec,rel", [("fp16x2", 3e-6), ("bf16x2", 2e-3)])
@pytest.mark.parametrize("nc,n_bins,n_det,n_sub", [(1, 3, 4, 1), (2, 50, 2, 15), (3, 65, 1, 16),
                                                   (5, 300, 3, 17), (8, 129, 1, 33)])
def test_hh_rows(prec, rel, nc, n_bins, n_det, n_sub):
    from paper_2507_16022_amd import dotpe
    rng = np.random.default_rng(nc)
    modes = MODES8[:nc]
    wl = W.make_workload(5, n_int=40, n_ext=9, n_bins=max(n_bins, 3), modes=W.MODES_22, dets="H", n_phi=4,
                         snr=10.0, mc_range=(10.0, 40.0), q_range=(0.3, 1.0), with_bank=False)
    h = rng.normal(size=(40, nc, n_bins)) + 1j * rng.normal(size=(40, nc, n_bins))
    r = rng.normal(size=(n_det, 3)) * 6e6
    D = rng.normal(size=(n_det, 3, 3))
    D = D + np.swapaxes(D, 1, 2)
    w = rng.uniform(0.5, 2.0, (n_det, n_bins))
    d = rng.normal(size=(n_det, n_bins)) + 1j * rng.normal(size=(n_det, n_bins))
    idx = rng.permutation(40)[:n_sub]
    ctx = dotpe.Context(0)
    bank = ctx.load_bank(h, modes, wl.f, precision=prec)
    ev = ctx.set_event(bank, d=d, w=w, det_r=r, det_D=D, ext=wl.ext, n_phi=4, sub_idx=idx)
    got = ev.eval_lnl(triples=True)["hh"]
    ev.close()
    bank.close()
    ctx.close()
    R, t = O.response(D, modes, wl.ext), O.arrival_times(r, wl.ext["lat"], wl.ext["lon"], wl.ext["t_geo"])
    m = np.array([mm for _, mm in modes], dtype=float)
    for q, i in enumerate(idx):
        _, hh = O.triple_inner_products(h[i], R, t, wl.f, m, O.phase_grid(4), d, w)
        # split operands and FP32 sums of up to 32 terms per output: relative to the terms' size
        size = np.einsum("kb,ekc,cb->e", w, np.abs(R) ** 2, np.abs(h[i]) ** 2)[:, None] * nc
        assert np.all(np.abs(got[q] - hh) <= rel * size), (q, np.max(np.abs(got[q] - hh) / size))
