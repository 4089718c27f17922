"""Relative-binning weights with 1 to 64 lanes per weight: two to a thousand points of the grid per node's
support, dense and scattered nodes, weights that do not fill a workgroup, against the plain sums."""
import numpy as np
import pytest

from oracle import oracle as O

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nc,n_det,n_full,n_nodes,even", [
    (1, 1, 2, 2, True), (2, 3, 70, 70, True), (3, 2, 200, 23, True), (3, 1, 900, 100, False), (5, 2, 1000, 41, True),
    (2, 2, 3000, 33, False), (1, 2, 5000, 21, True)])
def test_rb_lanes(nc, n_det, n_full, n_nodes, even):
    from paper_2507_16022_amd import dotpe
    rng = np.random.default_rng(n_full)

    def cx(*s):
        return rng.normal(size=s) + 1j * rng.normal(size=s)
    f = np.linspace(20.0, 200.0, n_full)
    idx = np.unique(np.linspace(0, n_full - 1, n_nodes).astype(np.int64)) if even else \
        np.sort(rng.permutation(n_full)[:n_nodes])
    d, h0, w, t0 = cx(n_det, n_full), cx(nc, n_full), rng.uniform(0.5, 2.0, (n_det, n_full)), rng.normal(size=n_det)
    ctx = dotpe.Context(0)
    w_dh, w_hh, dd = ctx.rb_weights(f, d, w, h0, idx, t0)
    ctx.close()
    a, b = O.rb_weights(f, d, w, h0, idx, t0)[:2]
    # rounding of up to 3000 terms, relative to the terms' size over the divisor
    for got, want in ((w_dh, a), (w_hh, b)):
        assert np.all(np.abs(got - want) <= 1e-12 * np.max(np.abs(want)))
    assert dd == pytest.approx(np.sum(w * np.abs(d) ** 2), rel=1e-12)
