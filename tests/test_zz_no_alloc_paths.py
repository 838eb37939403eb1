"""rexi_step_noalloc where its array holds the pole-per-lane schedule's boundary values whole or in part, and where
the tiled schedule takes the call, against the oracle and rexi_step."""
import numpy as np
import pytest

import synth
from tests.gpu_common import TOL, assert_parity, oracle_run_parallel

pytestmark = pytest.mark.gpu


# (T, S, M, nsteps, same): the 64 MiB array holds a slot for every workgroup (split and whole chains); between 512
# slots and the workgroups' number, so that workgroups take several items in turn (one and eight states); too few,
# so that the tiled schedule runs, whose sums are in another order.  plan_host's noalloc_routes says so on the CPU.
@pytest.mark.parametrize("T,S,M,nsteps,same", [(100, 1, 250, 2, True), (60, 1, 500, 2, True), (100, 1, 500, 2, True),
                                               (31, 8, 1000, 2, True), (60, 4, 500, 2, False), (150, 1, 250, 1, False)])
def test_noalloc_paths(T, S, M, nsteps, same):
    import torch
    import paper_1812_03431_amd as rexi
    print(f"\n[gpu] noalloc T={T} S={S} M={M}", flush=True)
    w = synth.Workload("noalloc", T=T, nlat=0, nlon=0, dt=1800.0, M=M, states=S)
    plan = rexi.plan_for(w, grid=False)
    u0 = synth.random_state(T, S, T + S)
    x = torch.from_numpy(u0).to("cuda:0")
    regular = plan.step(x, nsteps).cpu().numpy()
    assert plan.schedule_name(S, plan.chosen_schedule(S)).startswith("sweep")
    out = torch.full_like(x, float("nan"))
    got = plan.step_noalloc(x, nsteps, out=out).cpu().numpy()
    if same:
        assert np.array_equal(got, regular)
    else:
        assert_parity(got, regular, T, tol=TOL, what="noalloc and rexi_step")
    orders = sorted({0, 1, 2, T // 3, T // 2, T - 1, T})
    want = oracle_run_parallel(u0, w, nsteps, orders=orders, workers=1)
    assert_parity(got, want, T, orders=orders, tol=TOL, what="noalloc")
