"""Envelope maxima that are known from the bins without a second evaluation: stations without a signal, directions at
which the pattern is singular (a zero field), and traces that are not numbers; with infinite and overflowing ones, which
are evaluated.  Against the call that also returns the traces."""
import numpy as np
import pytest

from paper_1507_07733_amd import synth as S

from test_gpu_env_peaks import setup
from test_gpu_envelope import api  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [64, 32])
@pytest.mark.parametrize("n", [512, 1024, 2048, 4096])
def test_known_maxima(api, n, prec):  # noqa: F811
    import torch
    dirs = np.array([[40.0, 120.0], [90.0, 30.0], [12.0, 200.0]])      # the second: horizon, zero field
    volt = S.traces(9, n, cfg=4, event=n)
    volt[0] = 0.0
    volt[1] = np.nan
    volt[2, 0, 17] = np.nan
    volt[3, 1, n - 1] = np.inf
    volt[4, 0] = np.nan
    volt[5] *= 1e300 if prec == 64 else 1e36
    volt[6, 1] = 0.0
    full = dict(band_lo_hz=0, band_hi_hz=40_000_000)
    ident = S.identity_table(S.GRID_COARSE)
    for table, band in ((S.pattern_table(S.GRID_COARSE, cfg=0), {}), (ident, full),
                        (ident, dict(band_lo_hz=0, band_hi_hz=0))):
        print("[case] known maxima N", n, "prec", prec, band, flush=True)
        with np.errstate(over="ignore"):
            tab, ev, v = setup(api, prec, table, volt, **band)
        peak, arg, _ = api.unfold_envelope_scan(tab, ev, v, dirs)
        peak_t, arg_t, _ = api.unfold_envelope_scan(tab, ev, v, dirs, efield=True)
        torch.cuda.synchronize()
        assert bool((arg == arg_t).all())
        for st in range(9):
            same = torch.isclose(peak[:, st], peak_t[:, st], rtol=1e-12 if prec == 64 else 1e-5, atol=0, equal_nan=True)
            assert bool(same.all()), (st, peak[:, st], peak_t[:, st])
        assert not peak[:, 0].any() and not arg[:, 0].any()
        if table is not ident:
            assert not peak[1, [0, 6, 7, 8]].any() and bool(torch.isnan(peak[0, 1]).all())
