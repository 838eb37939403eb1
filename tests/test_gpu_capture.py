"""Steps captured into a caller's graph: replays stay right while the plan takes up other state counts."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


# register-resident, split and whole chains
@pytest.mark.parametrize("T,M", [(40, 20), (100, 20), (200, 150)])
def test_a_captured_step_outlives_the_growth_of_the_workspace(T, M):
    import torch
    import paper_1812_03431_amd as rexi
    print(f"\n[gpu] captured step T={T} M={M}", flush=True)
    w = synth.Workload("capture", T=T, nlat=0, nlon=0, dt=1800.0, M=M, states=8)
    plan = rexi.plan_for(w, grid=False)
    u = [torch.from_numpy(synth.random_state(T, 1, k)).to("cuda:0") for k in range(4)]
    want = [plan.step(x, 2).cpu().numpy() for x in u]
    src, out = u[0].clone(), torch.empty_like(u[0])
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        plan.step(src, 2, out=out)
    for k, S in enumerate((0, 2, 5, 8)):
        if S:
            more = torch.from_numpy(synth.random_state(T, S, 90 + S)).to("cuda:0")
            plan.step(more, 2)   # grows the shared buffers
            torch.full((1 << 24,), float("nan"), dtype=torch.float64, device="cuda:0")
        src.copy_(u[k])
        out.zero_()
        graph.replay()
        assert np.array_equal(out.cpu().numpy(), want[k]), (T, S)
