"""Envelope maxima and the one-event loop on both sides of the band widths from which the maxima come from the analytic
signals (a 48th of the samples in single precision, a 256th in double; in the loop a sixteenth), and of a quarter of
the samples.  The samples against the call that also returns the traces, the loop against the batched one."""
import numpy as np
import pytest

from paper_1507_07733_amd import synth as S

from helpers import TOL_FP32, TOL_FP64
from test_gpu_env_peaks import both, setup
from test_gpu_envelope import api  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [64, 32])
@pytest.mark.parametrize("n", [512, 1024, 2048, 4096])
def test_band_widths(api, n, prec):  # noqa: F811
    dirs = np.array([[40.0, 120.0], [70.0, 355.0]])
    pos = S.station_positions(12, area_km2=0.01 * n / 512)
    volt, _ = S.plane_wave_traces(pos, n, 15.0, 200.0, cfg=6, event=n)
    least = -(-n // (48 if prec == 32 else 256))
    for nb in (1, least - 1, least, least + 1, n // 16 - 1, n // 16, n // 4, n // 4 + 1):
        if nb < 1:
            continue
        k0 = n // 8
        band = dict(band_lo_hz=-(-k0 * S.FS_HZ // n), band_hi_hz=-(-(k0 + nb - 1) * S.FS_HZ // n))
        assert len(S.band_bins(n, S.FS_HZ, band["band_lo_hz"], band["band_hi_hz"])) == nb
        print("[case] band N", n, "prec", prec, "bins", nb, flush=True)
        tab, ev, v = setup(api, prec, S.identity_table(S.GRID_COARSE), volt, **band)
        peak, arg, peak_t = both(api, tab, ev, v, dirs)
        assert float(((peak - peak_t).abs() / peak_t).max()) <= (TOL_FP32 if prec == 32 else TOL_FP64)
        one = api.reconstruct(tab, ev, v, pos, max_iter=3, efield=True)
        many = api.reconstruct_batch(tab, ev, v.reshape(-1), [len(pos)], [0], pos, max_iter=3)[0]
        assert np.array_equal(one.times, many.times) and np.array_equal(one.dirs, many.dirs)
