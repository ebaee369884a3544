"""The one-event loop at 2048 and 4096 samples, a launch per pass (a workgroup per station, up to 256 stations, or 512
in single precision at 2048 samples): kept traces and maxima after convergence on both sides of these numbers; passes
that go out in several chunks and a loop that ends unconverged, or after one pass; and times that ties decide.  Against
the batched loop (the same directions and times to the bit), the oracle, and the single-direction call for the kept
traces."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_1507_07733_amd import synth as S

from helpers import TOL_FP32, TOL_FP64, assert_close, oracle_unfold
from test_gpu_envelope import api  # noqa: F401
from test_gpu_reconstruct import check_passes

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
@pytest.mark.parametrize("s,n", [(40, 4096), (256, 2048), (257, 2048), (256, 4096), (257, 4096), (512, 2048), (513, 2048),
                                 (1024, 4096)])
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


@pytest.mark.parametrize("prec", [64, 32])
@pytest.mark.parametrize("n", [2048, 4096])
@pytest.mark.parametrize("max_iter", [1, 2, 6, 7])
def test_loop_that_does_not_converge(api, n, max_iter, prec):  # noqa: F811
    """Noise: every pass the oracle's (double); single precision against the batched loop and the oracle's envelopes."""
    print("[case] recon pass noise N", n, "max_iter", max_iter, "prec", prec, flush=True)
    t = S.pattern_table(G, cfg=0)
    pos = S.station_positions(12, area_km2=6.0 * 12 / 124)
    volt = S.traces(12, n, cfg=0, event=900)
    tab, ev, v = setup(api, prec, t, volt)
    rec = api.reconstruct(tab, ev, v, pos, max_iter=max_iter, efield=True)
    equals_batch(api, tab, ev, v, pos, rec, max_iter)
    kept_results(api, tab, ev, v, rec, prec == 32)
    if prec == 64:
        dirs, times, conv = O.reconstruct(G, t, volt, pos, S.FS_HZ, S.BAND_LO_HZ, S.BAND_HI_HZ, max_iter=max_iter)
        assert len(dirs) == max_iter and not conv  # the case this test is for
        assert not rec.converged and np.array_equal(rec.times, times)
        assert np.max(np.abs(rec.dirs - dirs)) < 1e-9
    else:
        t, volt = t.astype(np.complex64), volt.astype(np.float32)
        check_passes(G, t, volt, pos, rec, TOL_FP32)
        ref, _, _ = oracle_unfold(G, t, volt, rec.direction[None, :])
        assert_close(rec.efield.cpu().numpy(), ref[0], True, "kept traces against the oracle")


@pytest.mark.parametrize("prec", [64, 32])
@pytest.mark.parametrize("n", [2048, 4096])
def test_times_decided_by_ties(api, n, prec):  # noqa: F811
    """Every station tied (traces of half the period), one station without a signal, one bin (a constant envelope), and
    a band from 0 Hz: the maxima that are evaluated again, each workgroup writing the coefficients it needs."""
    print("[case] recon pass ties N", n, "prec", prec, flush=True)
    s = 40
    pos = S.station_positions(s)
    volt, _ = S.plane_wave_traces(pos, n, 15.0, 200.0, cfg=6, event=n)
    half = volt.copy()
    half[..., n // 2:] = half[..., :n // 2]
    dead = volt.copy()
    dead[7] = 0.0
    pattern, ident = S.pattern_table(G, cfg=0), S.identity_table(G)
    for table, x, band in ((pattern, half, {}), (pattern, dead, {}),
                           (ident, volt, dict(band_lo_hz=50_000_000, band_hi_hz=50_000_000)),
                           (ident, volt + 3.0, dict(band_lo_hz=0, band_hi_hz=40_000_000))):
        tab, ev, v = setup(api, prec, table, x, **band)
        rec = api.reconstruct(tab, ev, v, pos, max_iter=4, efield=True)
        equals_batch(api, tab, ev, v, pos, rec, 4)
        kept_results(api, tab, ev, v, rec, prec == 32)
