"""The one-event loop at 2048 and 4096 samples, a launch per pass (a workgroup per station, up to 1024 stations): kept
traces and maxima after convergence with more stations than the device holds workgroups, and on both sides of the
1024 stations.  Against the batched loop (the same directions and times to the bit) and the single-direction call for
the kept traces."""
import numpy as np
import pytest

from paper_1507_07733_amd import synth as S

from helpers import TOL_FP32, TOL_FP64, assert_close
from test_gpu_envelope import api  # noqa: F401

pytestmark = pytest.mark.gpu
G = S.GRID_COARSE


def setup(api, prec, table, volt, **band):
    import torch
    f32 = prec == 32
    tab = api.Table(G, table.astype(np.complex64) if f32 else table)
    v = torch.from_numpy(np.ascontiguousarray(volt, dtype=np.float32 if f32 else np.float64)).cuda()
    ev = api.make_event(v.shape[0], v.shape[2], prec=api.AU_PREC_FP32 if f32 else api.AU_PREC_FP64,
                        trace_dtype=api.AU_F32 if f32 else api.AU_F64, **band)
    return tab, ev, v


def equals_batch(api, tab, ev, v, pos, rec, max_iter):
    one = api.reconstruct_batch(tab, ev, v.reshape(-1), [len(pos)], [0], pos, max_iter=max_iter)[0]
    assert np.array_equal(rec.dirs, one.dirs) and np.array_equal(rec.times, one.times)
    assert int(rec.converged) == one.converged


def kept_results(api, tab, ev, v, rec, f32):
    """The kept traces and maxima are those of the last direction."""
    z, a = rec.direction
    want = api.unfold_event(tab, ev, v, z, a).cpu().numpy()
    assert_close(rec.efield.cpu().numpy(), want, f32, "kept traces")
    peak, arg, _ = api.unfold_envelope_scan(tab, ev, v, rec.direction[None, :])
    assert np.array_equal(arg[0, :, 2].cpu().numpy(), rec.times[-1])
    assert float(((rec.peak - peak[0]).abs() / peak[0].clamp(min=1e-300 if not f32 else 1e-30)).max()) <= \
        (TOL_FP32 if f32 else TOL_FP64)


@pytest.mark.parametrize("prec", [64, 32])
@pytest.mark.parametrize("s,n", [(40, 4096), (700, 2048), (1024, 2048), (1025, 2048), (1024, 4096)])
def test_kept_traces_after_convergence(api, s, n, prec):  # noqa: F811
    import torch
    print("[case] recon pass S", s, "N", n, "prec", prec, flush=True)
    pos = S.station_positions(s)
    volt, _ = S.plane_wave_traces(pos, n, 20.0, 130.0, cfg=6, event=s)
    tab, ev, v = setup(api, prec, S.pattern_table(G, cfg=0), volt)
    out = torch.empty((s, 2, n), dtype=v.dtype, device="cuda")
    for _ in range(3):
        out.fill_(float("nan"))
        rec = api.reconstruct(tab, ev, v, pos, max_iter=12, efield=out)
        assert rec.converged
        equals_batch(api, tab, ev, v, pos, rec, 12)
        kept_results(api, tab, ev, v, rec, prec == 32)
