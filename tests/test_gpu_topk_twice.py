"""Top-k of a subset that names rows more than once: a pair is reported as often as its row is named, in one
block of equal records, whichever way the candidates are placed (counted up to 256, sorted beyond)."""
import numpy as np
import pytest

from synth import workload as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("times,rows,top_k", [(2, 5, 16), (7, 9, 64), (3, 200, 600), (40, 30, 100)])
def test_rows_named_twice(times, rows, top_k):
    from paper_2507_16022_amd import dotpe
    wl = W.config_tiny(seed=4, n_int=256, n_ext=64, snr=6.0)
    rng = np.random.default_rng(times)
    names = rng.permutation(256)[:rows]
    idx = rng.permutation(np.repeat(names, times)).astype(np.int64)
    ctx = dotpe.Context(0)
    bank = ctx.load_bank(wl.h, wl.modes, wl.f, wl.ln_w_int, precision="fp16x2")

    def top(sub, k):
        ev = ctx.set_event(bank, d=wl.d, w=wl.w, det_r=wl.det_r, det_D=wl.det_D, ext=wl.ext, n_phi=wl.n_phi,
                           ln_w_ext=wl.ln_w_ext, d_max=wl.d_max, d0=wl.d0, top_k=k, topk_window=1.5, sub_idx=sub)
        r = ev.evidence()
        again = ev.evidence()
        ev.close()
        for key in ("topk_i", "topk_e", "topk_o", "topk_lnp"):
            np.testing.assert_array_equal(r[key], again[key])
        return r
    once, many = top(names.astype(np.int64), top_k), top(idx, top_k)
    bank.close()
    ctx.close()
    n = min(len(once["topk_i"]) * times, top_k)
    print(f"{times} x {rows} rows: {len(once['topk_i'])} pairs within the window, {len(many['topk_i'])} reported")
    assert len(many["topk_i"]) == n == many["topk_count"] and n >= times
    for key in ("topk_i", "topk_e", "topk_o", "topk_lnp"):
        np.testing.assert_array_equal(many[key], np.repeat(once[key], times)[:n])
