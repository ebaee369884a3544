"""First station times of the reconstruction loop (the smallest sample maximising V_0^2 + V_1^2, in double), which the
spectrum kernel takes from the traces it transforms from 512 samples up (a kernel of their own below): equal to numpy's
for noise, for many equal maxima, for zero traces, and where samples are not numbers or infinite."""
import numpy as np
import pytest

from paper_1507_07733_amd import synth as S
from test_gpu_envelope import api  # noqa: F401

pytestmark = pytest.mark.gpu


def samples(kind, s, n, dtype):
    v = np.random.default_rng(n).standard_normal((s, 2, n))
    if kind == "ties":
        v = np.round(2 * v)
    if kind == "special":
        v[0] = 0.0
        v[1] = np.nan
        v[2, 0, :n // 2] = np.nan
        v[4, 0, 7] = np.inf
        v[5, 1, [9, n - 1]] = np.inf
    return v.astype(dtype)


@pytest.mark.parametrize("n", [256, 512, 1024, 2048, 4096])
@pytest.mark.parametrize("prec,dtype", [(64, np.float64), (32, np.float32), (32, np.float64), (64, np.float32)])
def test_first_times(api, n, prec, dtype):  # noqa: F811
    import torch
    print("[case] first times N", n, "prec", prec, dtype.__name__, flush=True)
    t = S.pattern_table(S.GRID_COARSE, cfg=0)
    tab = api.Table(S.GRID_COARSE, t if prec == 64 else t.astype(np.complex64))
    ev = api.make_event(3, n, prec=api.AU_PREC_FP64 if prec == 64 else api.AU_PREC_FP32,
                        trace_dtype=api.AU_F64 if dtype == np.float64 else api.AU_F32)
    ns = [3, 7, 40, 3]
    offs = np.cumsum([0] + ns[:-1]) * 2 * n
    pos = np.concatenate([S.station_positions(s) for s in ns])
    for kind in ("noise", "ties", "special"):
        v = samples(kind, sum(ns), n, dtype)
        res = api.reconstruct_batch(tab, ev, torch.from_numpy(v).cuda().reshape(-1), ns, offs, pos, max_iter=1)
        got = np.concatenate([r.times[0] for r in res])
        with np.errstate(all="ignore"):
            pw = v[:, 0].astype(np.float64) ** 2 + v[:, 1].astype(np.float64) ** 2
        assert np.array_equal(got, np.where(np.isnan(pw), -1.0, pw).argmax(axis=1)), kind
