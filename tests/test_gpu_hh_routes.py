"""The row-side (h|h) operand of banks with six to eight channels: one pass per detector of the 16-lane
sums, or a workgroup per row where that takes fewer rounds and the row fits LDS; both layouts, bins around
a chunk, rows too long for LDS, through the (h|h) of every triple."""
import numpy as np
import pytest

from oracle import oracle as O
from synth import workload as W

pytestmark = pytest.mark.gpu

MODES8 = ((2, 2), (2, 1), (3, 3), (3, 2), (4, 4), (3, 1), (4, 3), (4, 2))
MP8 = tuple((m, p) for m in (1, 2, 3, 4) for p in (0, 1))


@pytest.mark.parametrize("layout,nc,n_bins,n_det", [("lm", 6, 65, 2), ("mp", 6, 200, 3), ("mp", 8, 63, 2),
                                                    ("mp", 8, 256, 3), ("mp", 8, 1100, 3), ("mp", 8, 33, 8),
                                                    ("mp", 8, 1000, 8)])
def test_hh_many_channels(layout, nc, n_bins, n_det):
    from paper_2507_16022_amd import dotpe
    rng = np.random.default_rng(nc * n_det)
    chans = (MODES8 if layout == "lm" else MP8)[:nc]
    wl = W.make_workload(5, n_int=40, n_ext=7, n_bins=n_bins, modes=W.MODES_22, dets="H", n_phi=4, snr=10.0,
                         mc_range=(10.0, 40.0), q_range=(0.3, 1.0), with_bank=False)
    h = rng.normal(size=(40, nc, n_bins)) + 1j * rng.normal(size=(40, nc, n_bins))
    r = rng.normal(size=(n_det, 3)) * 6e6
    D = rng.normal(size=(n_det, 3, 3))
    D = D + np.swapaxes(D, 1, 2)
    w = rng.uniform(0.5, 2.0, (n_det, n_bins))
    d = rng.normal(size=(n_det, n_bins)) + 1j * rng.normal(size=(n_det, n_bins))
    idx = rng.permutation(40)[:19]
    ctx = dotpe.Context(0)
    bank = ctx.load_bank(h, chans, wl.f, precision="fp16x2", layout=layout)
    ev = ctx.set_event(bank, d=d, w=w, det_r=r, det_D=D, ext=wl.ext, n_phi=4, sub_idx=idx)
    got = ev.eval_lnl(triples=True)["hh"]
    ev.close()
    bank.close()
    ctx.close()
    R = O.response(D, chans, wl.ext) if layout == "lm" else O.response_mp(D, [p for _, p in chans], wl.ext)
    t = O.arrival_times(r, wl.ext["lat"], wl.ext["lon"], wl.ext["t_geo"])
    m = np.array([c[0] if layout == "mp" else c[1] for c in chans], dtype=float)
    for q, i in enumerate(idx):
        _, hh = O.triple_inner_products(h[i], R, t, wl.f, m, O.phase_grid(4), d, w)
        # split operands and FP32 sums of up to 32 terms per output: relative to the terms' size
        size = np.einsum("kb,ekc,cb->e", w, np.abs(R) ** 2, np.abs(h[i]) ** 2)[:, None] * nc
        assert np.all(np.abs(got[q] - hh) <= 3e-6 * size), (q, np.max(np.abs(got[q] - hh) / size))
