"""GPU parity of the pole-per-lane solve (schedules named "sweep") with the oracle, at the edges of its blocks of 12
chain elements, its batches of 64 poles and its tiles of up to 4 states."""
import numpy as np
import pytest

import synth
from oracle import rexi as orexi
from tests.gpu_common import A, OM, PB, TOL, assert_parity, oracle_coeffs

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _announce(request):
    import torch
    assert torch.cuda.is_available(), "no GPU"
    torch.zeros(1, device="cuda:0")
    print(f"\n[gpu] {request.node.nodeid}", flush=True)


def _gpu(x):
    import torch
    return torch.from_numpy(np.ascontiguousarray(x)).to("cuda:0")


# (T, S, M): chains up to T elements (+ a dummy) around 1, 2, 4, 12, 24 and 36; N = 2 (M + 11) + 1 poles just below and
# above 64 and 128; 1 to 9 states (tiles 1, 2, 3, 4, 2+3, 3+3, 3+3+3).  From 24 elements on chains are split between
# two waves; up to 16 pairs a half it stays in registers (T = 63 .. 65 on both sides of that).
@pytest.mark.parametrize("T,S,M", [(26, 5, 20), (31, 1, 52), (48, 2, 20), (49, 3, 21), (63, 2, 20), (64, 1, 52), (65, 4, 20),
                                   (1, 1, 8), (2, 3, 20), (3, 2, 21), (4, 5, 20), (11, 4, 52), (12, 1, 53), (13, 9, 21),
                                   (23, 2, 52), (24, 6, 53), (25, 1, 21), (37, 3, 52)])
def test_sweep_edges(T, S, M):
    import paper_1812_03431_amd as rexi
    dt = 0.5 * 0.2 * M / (np.sqrt(PB * T * (T + 1)) / A)   # half of the covered range
    dt = min(dt, 7200.0)
    w = synth.Workload("sweep", T=T, nlat=0, nlon=0, dt=dt, M=M, states=S)
    u0 = synth.random_state(T, S, 700 + T)
    co = oracle_coeffs(M, w.h, w.L)
    want = orexi.rexi_run(u0, 2, T, dt, co, A, OM, PB)
    want_a = orexi.rexi_run(u0, 1, T, dt, co, A, OM, PB, adjoint=True)
    plan = rexi.plan_for(w, grid=False)
    names = [plan.schedule_name(S, i) for i in range(plan.schedule_count(S))]
    assert names[plan.chosen_schedule(S)].startswith("sweep")
    for i, name in enumerate(names):
        if "sweep" not in name:
            continue
        plan.set_schedule(S, i)
        assert_parity(plan.step(_gpu(u0), 2).cpu().numpy(), want, T, tol=TOL, what=f"{name} T{T} S{S}")
        assert_parity(plan.step_adjoint(_gpu(u0)).cpu().numpy(), want_a, T, tol=TOL, what=f"{name} adjoint T{T} S{S}")


def test_without_coriolis_the_tiled_schedules_run():
    # the pole-per-lane form scales by the Coriolis couplings, so it is not offered where there are none
    import paper_1812_03431_amd as rexi
    T, S, M, dt = 14, 2, 32, 3600.0
    w = synth.Workload("still", T=T, nlat=0, nlon=0, dt=dt, M=M, states=S)
    p = rexi.params_for(w, grid=False)
    p.omega = 0.0
    plan = rexi.Plan(p)
    assert not any("sweep" in plan.schedule_name(S, i) for i in range(plan.schedule_count(S)))
    u0 = synth.random_state(T, S, 31)
    want = orexi.rexi_run(u0, 1, T, dt, oracle_coeffs(M, w.h, w.L), A, 0.0, PB)
    assert_parity(plan.step(_gpu(u0)).cpu().numpy(), want, T, what="omega 0")


def test_a_non_finite_state_stays_in_its_state_and_order():
    # NaN in one order of one state: the other states and orders are as without it
    import paper_1812_03431_amd as rexi
    T, S = 20, 3
    w = synth.Workload("nan", T=T, nlat=0, nlon=0, dt=3600.0, M=32, states=S)
    u0 = synth.random_state(T, S, 41)
    plan = rexi.plan_for(w, grid=False)
    ref = plan.step(_gpu(u0)).cpu().numpy()
    m, n = 5, 9
    i = m * (T + 1) - m * (m - 1) // 2 + (n - m)
    u0[1, 1, i] = np.nan
    got = plan.step(_gpu(u0)).cpu().numpy()
    lo = m * (T + 1) - m * (m - 1) // 2
    same = np.ones(got.shape, dtype=bool)
    same[1, :, lo:lo + T + 1 - m] = False
    assert np.array_equal(got[same], ref[same])
    assert np.isnan(got[1, 1, i])
