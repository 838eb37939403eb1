"""The f-sphere kernel at the edges of its degree tiles, pole passes and pair
chunks, against the oracle."""
import numpy as np
import pytest

import synth
from oracle import rexi as orexi
from tests.gpu_common import A, OM, PB, assert_parity, oracle_coeffs

pytestmark = pytest.mark.gpu


# (M h above the largest dt w_n, so that every entry of the propagator is an
# approximation and not the rounding noise of a vanishing sum); eight degrees to a workgroup, 64 poles (N = 2 (M + 11) + 1) to a pass, 64
# (state, order) pairs to a pass of a workgroup
@pytest.mark.parametrize("T,S,M", [(1, 1, 8), (7, 2, 20), (8, 9, 21), (15, 4, 64), (16, 64, 32), (23, 3, 9), (130, 5, 80)])
@pytest.mark.parametrize("adjoint", [False, True])
def test_fsphere_tile_edges(T, S, M, adjoint):
    import torch
    import paper_1812_03431_amd as rexi
    print(f"\n[gpu] fsphere T={T} S={S} M={M} adjoint={adjoint}", flush=True)
    f0 = synth.FSPHERE_F0
    w = synth.Workload("fs", T=T, nlat=0, nlon=0, dt=1800.0, M=M, states=S)
    plan = rexi.plan_for(w, max_states=S, grid=False, fsphere=f0)
    u = synth.random_state(T, S, T + S)
    x = torch.from_numpy(u).to("cuda:0")
    got = (plan.step_adjoint if adjoint else plan.step)(x, 2).cpu().numpy()
    co = oracle_coeffs(w.M, w.h, w.L)
    want = u
    for _ in range(2):
        want = orexi.rexi_step(want, T, w.dt, co, A, OM, PB, adjoint=adjoint, fsphere=f0)
    assert_parity(got, want, T, what=f"f-sphere T{T} S{S} M{M}")
