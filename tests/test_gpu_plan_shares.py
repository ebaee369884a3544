"""Double-precision plans, whose unfold stage takes equal shares of the work per workgroup: classes of one
station-unfold (most shares empty), of fewer than one round of stations per workgroup, of rows cut in the middle, and
of several pieces per share; in list order and by XCD; before and after the tuner has changed the shapes.  Against the
one-event scan of the same shape (the same operations in the same order: equal bits), and after tuning to rounding."""
import numpy as np
import pytest

from paper_1507_07733_amd import synth as S

from test_gpu_envelope import api  # noqa: F401

pytestmark = pytest.mark.gpu
G = S.GRID_COARSE


@pytest.mark.parametrize("flags", [0, 4, 7])
def test_every_station_once(api, flags):  # noqa: F811
    import torch
    tab = api.Table(G, S.pattern_table(G, cfg=0))
    specs = [(1, 512, [[40.0, 10.0]]),                                                          # one unfold
             (7, 256, S.direction_grid(7, 3)), (9, 256, [[30.0, 200.0]]), (40, 256, S.direction_grid(32, 64)),
             (2, 64, S.direction_grid(1, 3)), (77, 64, S.direction_grid(2, 2)),                 # rows of padded rounds
             (61, 2048, S.direction_grid(3, 11)), (1, 2048, [[88.0, 0.0]]),
             (124, 4096, S.direction_grid(4, 4)), (33, 1024, S.direction_grid(16, 8))]
    plan = api.Plan(tab, specs, prec=api.AU_PREC_FP64, trace_dtype=api.AU_F64, flags=flags)
    volt = np.zeros(plan.volt_elems)
    want = []
    for e, (s, n, d) in enumerate(specs):
        v = S.traces(s, n, cfg=1, event=300 + e)
        volt[plan.volt_offsets[e]:plan.volt_offsets[e] + v.size] = v.ravel()
        ev = api.make_event(s, n, prec=api.AU_PREC_FP64, trace_dtype=api.AU_F64)
        want.append(api.unfold_direction_scan(tab, ev, torch.from_numpy(v).cuda(), d))
    dv = torch.from_numpy(volt).cuda()
    out = torch.empty(plan.efield_elems, dtype=torch.float64, device="cuda")
    for rep in range(3):
        print("[case] plan shares flags", flags, "run", rep, flush=True)
        out.fill_(float("nan"))
        plan.run(dv, out)
        torch.cuda.synchronize()
        for e in range(len(specs)):
            assert torch.equal(plan.event_output(out, e), want[e]), (rep, specs[e][:2])
    plan.autotune(dv, out, reps=1)
    out.fill_(float("nan"))
    plan.run(dv, out)
    torch.cuda.synchronize()
    for e in range(len(specs)):
        # another shape orders the butterflies' products differently: a few ulp per pass
        err = (plan.event_output(out, e) - want[e]).abs().max()
        assert err <= 1e-12 * want[e].abs().max(), specs[e][:2]
