"""The one-launch single-direction call at 256, 512 and 1024 samples (half a wavefront to two per transform, with an
even and an odd number of exchanges) against the three launches of a one-direction scan, to rounding, and the oracle;
one station and an odd number of them, bands from DC, of one bin and empty, the wrap, the zenith and the horizon."""
import numpy as np
import pytest

from paper_1507_07733_amd import synth as S

from helpers import assert_close, oracle_unfold
from test_gpu_envelope import api  # noqa: F401

pytestmark = pytest.mark.gpu
G = S.GRID_COARSE


@pytest.mark.parametrize("prec", [64, 32])
@pytest.mark.parametrize("n", [256, 512, 1024])
def test_one_launch_short_traces(api, n, prec):  # noqa: F811
    import torch
    f32 = prec == 32
    dt = np.float32 if f32 else np.float64
    bands = [(S.pattern_table(G, cfg=0), {}), (S.identity_table(G), dict(band_lo_hz=0, band_hi_hz=40_000_000)),
             (S.identity_table(G), dict(band_lo_hz=50_000_000, band_hi_hz=50_000_000)),
             (S.identity_table(G), dict(band_lo_hz=41_000_000, band_hi_hz=41_010_000))]
    for t, band in bands:
        tt = t.astype(np.complex64) if f32 else t
        tab = api.Table(G, tt)
        for s in (1, 33):
            print("[case] one launch N", n, "prec", prec, band, "S", s, flush=True)
            v = (S.traces(s, n, cfg=1, event=n + s) + 1.5).astype(dt)
            ev = api.make_event(s, n, prec=api.AU_PREC_FP32 if f32 else api.AU_PREC_FP64,
                                trace_dtype=api.AU_F32 if f32 else api.AU_F64, **band)
            dv = torch.from_numpy(v).cuda()
            for z, a in ((37.5, 211.0), (0.0, 359.9), (88.0, -30.0), (90.0, 10.0)):
                c1 = torch.zeros(2, dtype=torch.int64, device="cuda")
                c3 = torch.zeros_like(c1)
                one = api.unfold_event(tab, ev, dv, z, a, counts=c1).cpu().numpy()
                three = api.unfold_direction_scan(tab, ev, dv, [[z, a]], counts=c3)[0].cpu().numpy()
                assert torch.equal(c1, c3)
                scale = np.abs(three).max(axis=(1, 2))
                err = np.abs(one.astype(np.float64) - three).max(axis=(1, 2))
                assert np.all(err <= (1e-6 if f32 else 1e-13) * scale), (z, a)
                if not band and z < 80.0:
                    ref, _, _ = oracle_unfold(G, tt, v, [[z, a]])
                    assert_close(one, ref[0], f32, "one launch")
