"""Orders past nlon / 2, whose bins alias, at the FFT lengths where only truncations above 40 have them (T is at most
1023, so nlon = 1024 is the longest), against the oracle."""
import numpy as np
import pytest

import synth
from oracle import sh as osh

pytestmark = pytest.mark.gpu

TOL = 5e-12   # as for the flat spectra of the other transform tests


# the first order past nlon / 2, some more, and all there are; few latitudes (the sums over
# latitudes and degrees are the same on both sides, whether or not they resolve the orders)
@pytest.mark.parametrize("nlon", [128, 256, 512, 1024])
@pytest.mark.parametrize("past", [0, 1, 37, -1])
def test_aliased_orders_match_oracle(nlon, past):
    import torch
    import paper_1812_03431_amd as rexi
    T, nlat, B = (nlon - 1 if past < 0 else nlon // 2 + past), 10, 3
    print(f"\n[gpu] aliased fft nlon={nlon} T={T}", flush=True)
    w = synth.Workload("sh", T=T, nlat=nlat, nlon=nlon, dt=3600.0, M=8, states=1)
    plan = rexi.plan_for(w, max_fields=B)
    rng = np.random.default_rng(nlon + past)
    spec = rng.standard_normal((B, plan.nspec)) + 1j * rng.standard_normal((B, plan.nspec))
    spec[:, :T + 1] = spec[:, :T + 1].real
    want = osh.synthesis(spec, T, nlat, nlon)
    got = plan.sh_inverse(torch.from_numpy(spec).to("cuda:0")).cpu().numpy()
    assert np.max(np.abs(got - want)) / np.max(np.abs(want)) < TOL
    grid = rng.standard_normal((B, nlat, nlon))
    want = osh.analysis(grid, T)
    got = plan.sh_forward(torch.from_numpy(grid).to("cuda:0")).cpu().numpy()
    assert np.max(np.abs(got - want)) / np.max(np.abs(want)) < TOL
