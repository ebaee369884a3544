"""Double-precision scans on both sides of the direction count from which spectra and coefficients take a launch each
(three quarters of 2^20 directions x samples), against a plan of the same event."""
import numpy as np
import pytest

from paper_1507_07733_amd import synth as S

from test_gpu_envelope import api  # noqa: F401

pytestmark = pytest.mark.gpu
G = S.GRID_COARSE


@pytest.mark.parametrize("n", [512, 1024, 2048, 4096])
def test_scan_at_the_line(api, n):  # noqa: F811
    import torch
    tab = api.Table(G, S.pattern_table(G, cfg=0))
    every = S.direction_grid(50, 41)
    v = S.traces(3, n, cfg=1, event=n)
    dv = torch.from_numpy(v).cuda()
    ev = api.make_event(3, n)
    for d in ((3 << 18) // n, (3 << 18) // n + 1):
        print("[case] scan line N", n, "D", d, flush=True)
        c1, c2 = (torch.zeros(2, dtype=torch.int64, device="cuda") for _ in range(2))
        got = api.unfold_direction_scan(tab, ev, dv, every[:d], counts=c1)
        plan = api.Plan(tab, [(3, n, every[:d])], prec=api.AU_PREC_FP64, trace_dtype=api.AU_F64)
        want = torch.empty(plan.efield_elems, dtype=got.dtype, device="cuda")
        plan.run(dv, want, c2)
        assert torch.equal(c1, c2)
        assert (got - plan.event_output(want, 0)).abs().max() <= 1e-13 * want.abs().max()
