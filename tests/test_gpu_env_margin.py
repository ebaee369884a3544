"""Envelope maxima with and without traces, on signals whose envelopes are flat or whose rounding is large against them:
swept sines, chirps, a carrier 10^4 times its noise, two tones.  The samples are equal, and the maxima are within half
of the 32 u (of the total field's maximum) inside which samples are decided again."""
import numpy as np
import pytest

from paper_1507_07733_amd import synth as S

from test_gpu_env_peaks import both, setup
from test_gpu_envelope import api  # noqa: F401

pytestmark = pytest.mark.gpu


def signals(n, s, r):
    t = np.arange(n) / S.FS_HZ
    ph = r.uniform(0, 2 * np.pi, (3, s, 2, 1))
    f0, f1 = r.uniform(35e6, 45e6, (s, 2, 1)), r.uniform(60e6, 75e6, (s, 2, 1))
    yield "sweep", np.sin(2 * np.pi * (f0 * t + (f1 - f0) * t * t * S.FS_HZ / (2 * n)) + ph[0])
    yield "tones", np.sin(2 * np.pi * 40.1e6 * t + ph[0]) + np.sin(2 * np.pi * 71.3e6 * t + ph[1])
    carrier = round(55e6 * n / S.FS_HZ) * S.FS_HZ / n
    yield "carrier", np.sin(2 * np.pi * carrier * t + ph[2]) + 1e-4 * r.standard_normal((s, 2, n))
    kb = S.band_bins(n)
    z = np.zeros((s, 2, n // 2 + 1), dtype=complex)
    z[..., kb] = np.exp(1j * (np.pi * np.arange(len(kb)) ** 2 * r.uniform(0.2, 1.0, (s, 2, 1)) / len(kb) + ph[0]))
    yield "chirp", np.fft.irfft(z, n=n) * n / len(kb)


@pytest.mark.parametrize("prec", [64, 32])
@pytest.mark.parametrize("n", [512, 1024, 2048, 4096])
def test_evaluations_within_half_the_margin(api, n, prec):  # noqa: F811
    r = np.random.default_rng(n)
    dirs = np.stack([r.uniform(0, 87, 120), r.uniform(0, 360, 120)], axis=1)
    u = 2.0 ** (-24 if prec == 32 else -53)
    for name, volt in signals(n, 60, r):
        print("[case] env margin N", n, "prec", prec, name, flush=True)
        tab, ev, v = setup(api, prec, S.pattern_table(S.GRID_COARSE, cfg=0), volt)
        peak, _, peak_t = both(api, tab, ev, v, dirs)
        off = (peak.double() - peak_t.double()).abs() / peak_t[..., 2:].double() / u
        assert float(off.max()) <= 16.0, name
