"""The row-side (h|h) sums of long rows (more than 64 KB of amplitudes and weights) take the split bank's
values whole: hi + lo can span more bits than a float holds.  One channel constant, the other with a sum over the bins that nearly vanishes, so that S_1 is the
small remainder of values of order one; hh(0) - hh(pi) = 4 Re S_1 without S_0's rounding."""
import numpy as np
import pytest

from oracle import oracle as O
from synth import workload as W

pytestmark = pytest.mark.gpu


def _split(x):
    """The bank's FP16 hi + lo of x, as stored (largest component in [2^13, 2^14)), in double."""
    sc = 2.0 ** (np.floor(np.log2(np.max(np.abs(x)))) - 13)
    hi = (x / sc).astype(np.float16)
    lo = (x / sc - hi.astype(np.float64)).astype(np.float16)
    return (hi.astype(np.float64) + lo.astype(np.float64)) * sc


@pytest.mark.parametrize("n_bins", [3000, 4001])
def test_hh_rows_take_every_bit(n_bins):
    from paper_2507_16022_amd import dotpe
    rng = np.random.default_rng(n_bins)
    modes, n = ((2, 2), (2, 1)), 17
    wl = W.make_workload(5, n_int=1, n_ext=6, n_bins=n_bins, modes=W.MODES_22, dets="H", n_phi=2, snr=10.0,
                         mc_range=(10.0, 40.0), q_range=(0.3, 1.0))
    # values of up to 24 bits below one, the largest 1.5 in every row
    h = np.full((n, 2, n_bins), 1.0, dtype=complex)
    h[:, 1] = np.round(rng.uniform(-1, 1, (n, n_bins)) * 2.0 ** 24) / 2.0 ** 24
    h[:, 1, 0] = 1.5
    for i in range(n):
        for _ in range(50):              # (kept of order one: the remainder spread over the bins)
            h[i, 1, 1:] -= np.sum(h[i, 1].real) / (n_bins - 1)
        h[i, 1, 1:] = np.round(h[i, 1, 1:].real * 2.0 ** 24) / 2.0 ** 24
    w = np.ones((1, n_bins))
    D, r = wl.det_D[:1], wl.det_r[:1]
    ctx = dotpe.Context(0)
    bank = ctx.load_bank(h, modes, wl.f, precision="fp16x2")
    ev = ctx.set_event(bank, d=np.ones((1, n_bins), dtype=complex), w=w, det_r=r, det_D=D, ext=wl.ext, n_phi=2)
    hh = ev.eval_lnl(triples=True)["hh"]
    ev.close()
    bank.close()
    ctx.close()
    R = O.response(D, modes, wl.ext)                       # [e, k, c]
    q = R[:, 0, 0] * np.conj(R[:, 0, 1])
    for i in range(n):
        v = _split(h[i].real)
        s1 = np.sum(v[0] * v[1]) * q
        # the row operand's outputs keep 2^-38 of its largest one (sum h_22^2 = n_bins), and both operands 2^-22
        # of S_1 itself; twice that
        tol = 4 * (2.0 ** -37 * n_bins * (np.abs(q.real) + np.abs(q.imag)) + 2.0 ** -20 * np.abs(s1))
        err = np.abs((hh[i, :, 0] - hh[i, :, 1]) - 4 * s1.real)
        assert np.all(err <= tol), (i, np.max(err / tol))
