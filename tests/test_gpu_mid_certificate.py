"""Events of 256 to 2047 tiles of 128 x 128 with a small cut: where the certificate decides how many passes
an event takes, it is as tight, and the passes as few, as with the fast pass."""
import pytest

from synth import workload as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp16x2", "bf16x2"])
@pytest.mark.parametrize("delta", [4.0, 8.0])
def test_small_cut(prec, delta):
    from paper_2507_16022_amd import dotpe
    wl = W.make_workload(3, n_int=4096, n_ext=1030, n_bins=64, modes=W.MODES_HM, dets="HL", n_phi=16, snr=15.0,
                         mc_range=(10.0, 40.0), q_range=(0.3, 1.0))
    ctx = dotpe.Context(0)
    bank = ctx.load_bank(wl.h, wl.modes, wl.f, wl.ln_w_int, precision=prec)

    def evidence(target, flags):
        ev = ctx.set_event(bank, d=wl.d, w=wl.w, det_r=wl.det_r, det_D=wl.det_D, ext=wl.ext, n_phi=16,
                           ln_w_ext=wl.ln_w_ext, d_max=wl.d_max, d0=wl.d0, cut_delta=delta, cut_target=target,
                           flags=flags)
        r = ev.evidence()
        ev.close()
        return r
    fast = evidence(1e3, dotpe.FLAG_NO_BOUND_PASS)
    wide = fast["ln_z_upper"] - fast["ln_z"]
    assert fast["n_passes"] == 1 and wide > 0.0
    # a target that the fast pass just meets
    r = evidence(1.1 * wide, 0)
    bank.close()
    ctx.close()
    print(f"{prec} cut {delta}: certificate {wide:.3g}, {r['n_passes']} passes, {r['ln_z_upper'] - r['ln_z']:.3g}")
    for k in ("n_passes", "cut_delta_used", "n_tiles_rerun", "n_pairs_bounded", "ln_z", "ln_z_upper"):
        assert r[k] == fast[k], k
