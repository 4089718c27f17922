"""Posterior draws at the edges of the tiles they are resolved in: one pair, partial tiles, more
draws than pairs, many draws of one tile, both tile shapes (64 x 64 split precisions, 64 x 32
FP64).  The expected draws are formed from the library's own per-pair ln L (dotpe_eval_lnl), in
the tile order; a draw within rounding of a boundary may land on either side."""
import numpy as np
import pytest

from oracle import oracle as O
from synth import workload as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,tn", [("fp16x2", 64), ("fp64", 32)])
@pytest.mark.parametrize("n_i,n_e,n_s", [(1, 1, 5), (65, 1, 200), (64, 64, 1), (70, 131, 3000)])
def test_draws_at_tile_edges(prec, tn, n_i, n_e, n_s):
    from paper_2507_16022_amd import dotpe
    wl = W.config_tiny(seed=8, snr=5.0).subset(rows=np.arange(n_i), cols=np.arange(n_e))
    ctx = dotpe.Context(0)
    bank = ctx.load_bank(wl.h, wl.modes, wl.f, wl.ln_w_int, precision=prec)
    ev = ctx.set_event(bank, d=wl.d, w=wl.w, det_r=wl.det_r, det_D=wl.det_D, ext=wl.ext,
                       n_phi=wl.n_phi, ln_w_ext=wl.ln_w_ext, d_max=wl.d_max, d0=wl.d0)
    lnp = ev.eval_lnl()["lnl"] + wl.ln_w_int[:, None] + wl.ln_w_ext[None, :]
    ev.evidence()
    g = ev.sample_posterior(n_samples=n_s, u0=0.25, seed=3)
    order = [(i, e) for a in range(0, n_i, 64) for b in range(0, n_e, tn)
             for i in range(a, min(a + 64, n_i)) for e in range(b, min(b + tn, n_e))]
    w = np.exp(np.array([lnp[p] for p in order]) - lnp.max())
    cum = np.cumsum(w) / np.sum(w)
    pos = {p: k for k, p in enumerate(order)}
    expect = O.systematic_draws(w, n_s, 0.25)
    got = np.array([pos[(int(i), int(e))] for i, e in zip(g["i"], g["e"])])
    # FP32 phase sums: the pairs' weights agree to ~1e-6 relative
    for s in np.flatnonzero(got != expect):
        lo = cum[got[s] - 1] if got[s] else 0.0
        assert lo - 2e-6 <= (s + 0.25) / n_s <= cum[got[s]] + 2e-6, s
    assert np.mean(got == expect) >= 0.99
    assert np.max(np.abs(g["ln_p_pair"] - [lnp[order[k]] for k in got])) < 1e-5
    assert np.all((g["distance"] > 0) & (g["distance"] <= wl.d_max))
    assert np.all((g["o"] >= 0) & (g["o"] < wl.n_phi))
    ev.close()
    bank.close()
    ctx.close()
