"""Double-precision plans tuned while their work lists are in use: a graph captured before the tuning, from a shape that
the tuner leaves, replays with the lists it was captured with, as do runs still in flight on another stream."""
import numpy as np
import pytest

from paper_1507_07733_amd import synth as S

from test_gpu_envelope import api  # noqa: F401

pytestmark = pytest.mark.gpu
G = S.GRID_COARSE
SPECS = [(61, 2048, S.direction_grid(3, 11)), (7, 256, S.direction_grid(7, 3)), (124, 4096, S.direction_grid(4, 4)),
         (33, 1024, S.direction_grid(16, 8)), (1, 2048, [[88.0, 0.0]])]


@pytest.mark.parametrize("flags", [0, 4])
def test_lists_in_use_survive_tuning(api, flags):  # noqa: F811
    import torch
    tab = api.Table(G, S.pattern_table(G, cfg=0))
    lengths = (256, 1024, 2048, 4096)
    was = [api.get_unfold_variant(api.AU_PREC_FP64, n) for n in lengths]
    try:
        for n in lengths:
            api.set_unfold_variant(api.AU_PREC_FP64, n, 0)
        plan = api.Plan(tab, SPECS, prec=api.AU_PREC_FP64, trace_dtype=api.AU_F64, flags=flags)
    finally:
        for n, v in zip(lengths, was):
            api.set_unfold_variant(api.AU_PREC_FP64, n, v)
    volt = np.zeros(plan.volt_elems)
    for e, (s, n, _) in enumerate(SPECS):
        v = S.traces(s, n, cfg=1, event=300 + e)
        volt[plan.volt_offsets[e]:plan.volt_offsets[e] + v.size] = v.ravel()
    dv = torch.from_numpy(volt).cuda()
    want, out, tuned = (torch.full((plan.efield_elems,), float("nan"), dtype=torch.float64, device="cuda")
                        for _ in range(3))
    plan.run(dv, want)
    torch.cuda.synchronize()
    assert torch.isfinite(want).all()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        plan.run(dv, out)
    side = torch.cuda.Stream()
    for rep in range(3):
        print("[case] tuned plan flags", flags, "run", rep, flush=True)
        ahead = torch.full_like(want, float("nan"))
        torch.cuda.synchronize()
        with torch.cuda.stream(side):       # these runs may still be going on when the tuner starts
            for _ in range(20):
                plan.run(dv, ahead)
        plan.autotune(dv, tuned, reps=1)
        torch.cuda.synchronize()
        assert (ahead - want).abs().max() <= 1e-12 * want.abs().max()   # (the later repeats: the tuned shape)
        out.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want)       # the shape it was captured with, so the same bits
        tuned.fill_(float("nan"))
        plan.run(dv, tuned)
        torch.cuda.synchronize()
        assert (tuned - want).abs().max() <= 1e-12 * want.abs().max()
    graph.reset()
