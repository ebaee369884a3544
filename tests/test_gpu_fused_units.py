"""Fused plans of few stations, whose units are cut to single stations and parts of their directions (also uneven ones
and of one direction), and of enough stations for two and for four or eight stations a unit, in list order and by XCD:
every trace written, against the one-event scan.  Single-precision bound: the two kernels' products contract apart."""
import numpy as np
import pytest

from paper_1507_07733_amd import synth as S

from test_gpu_envelope import api  # noqa: F401

pytestmark = pytest.mark.gpu
G = S.GRID_COARSE


@pytest.mark.parametrize("flags", [0, 7])
@pytest.mark.parametrize("n", [2048, 4096])
@pytest.mark.parametrize("specs", [[(1, 64)], [(3, 7), (1, 1), (5, 63)], [(124, 2)] * 5, [(124, 1)] * 40, [(61, 3)] * 80])
def test_every_trace_of_a_fused_plan(api, specs, n, flags):  # noqa: F811
    import torch
    tab = api.Table(G, S.pattern_table(G, cfg=0).astype(np.complex64))
    dirs = S.direction_grid(8, 8)
    plan = api.Plan(tab, [(s, n, dirs[:d]) for s, d in specs], prec=api.AU_PREC_FP32, trace_dtype=api.AU_F32,
                    flags=flags | api.AU_PLAN_FUSED)
    print("[case] fused units", specs[:3], len(specs), "N", n, "flags", flags, flush=True)
    base = S.traces(124, n, cfg=1, event=17, dtype=np.float32)
    volt = torch.zeros(plan.volt_elems, dtype=torch.float32, device="cuda")
    for e, (s, _) in enumerate(specs):
        v = torch.from_numpy(np.roll(base, e, axis=0)[:s].copy()).cuda()
        volt[plan.volt_offsets[e]:plan.volt_offsets[e] + v.numel()] = v.ravel()
    out = torch.full((plan.efield_elems,), float("nan"), dtype=torch.float32, device="cuda")
    plan.run(volt, out)
    plan.run(volt, out)
    torch.cuda.synchronize()
    for e, (s, d) in enumerate(specs):
        ev = api.make_event(s, n, prec=api.AU_PREC_FP32, trace_dtype=api.AU_F32)
        v = volt[plan.volt_offsets[e]:plan.volt_offsets[e] + s * 2 * n].reshape(s, 2, n)
        want = api.unfold_direction_scan(tab, ev, v, dirs[:d])
        err = (plan.event_output(out, e) - want).abs().amax(dim=(2, 3)) / want.abs().amax(dim=(2, 3))
        assert err.max() <= 2e-6, (e, s, d)
