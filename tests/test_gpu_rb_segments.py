"""Relative-binning weights at the edges of the sums: neighbouring nodes one point apart, spans of
63, 64 and 65 points (the lanes of a wave), nodes inside the grid's ends, one channel and detector,
and (d|d) over more data than one block sums."""
import numpy as np
import pytest

from oracle import oracle as O

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,C,F,nodes", [
    (1, 1, 2, [0, 1]), (2, 3, 400, [3, 4, 67, 131, 196, 390]), (3, 5, 262147, [0, 1000, 262146]),
])
def test_rb_weight_spans(K, C, F, nodes):
    from paper_2507_16022_amd import dotpe
    rng = np.random.default_rng(F)
    f = 20.0 + np.arange(F) * (100.0 / F)
    z = lambda *s: rng.normal(size=s) + 1j * rng.normal(size=s)
    d, h0, w = z(K, F), z(C, F), rng.uniform(0.1, 2.0, (K, F))
    t0 = rng.uniform(-0.01, 0.01, K)
    ctx = dotpe.Context(0)
    wdh, whh, dd = ctx.rb_weights(f, d, w, h0, np.array(nodes), t0)
    ctx.close()
    # sums of up to 2^18 terms in double precision, cancelling by up to ~1e3
    if F < 1000:
        rdh, rhh, rdd = O.rb_weights(f, d, w, h0, np.array(nodes), t0)
        assert np.max(np.abs(wdh - rdh)) <= 1e-11 * np.max(np.abs(rdh))
        assert np.max(np.abs(whh - rhh)) <= 1e-11 * np.max(np.abs(rhh))
    else:
        s = np.interp(np.arange(F), nodes, [0.0, 1.0, 0.0])
        ref = np.sum(w[1] * s * h0[2] * np.conj(h0[4])) / (h0[2, 1000] * np.conj(h0[4, 1000]))
        assert abs(whh[1, 2, 4, 1] - ref) <= 1e-9 * np.sum(w[1] * s * np.abs(h0[2] * h0[4])) / abs(h0[2, 1000] * h0[4, 1000])
        rdd = O.data_inner(d, w)
    assert dd == pytest.approx(rdd, rel=1e-12)
