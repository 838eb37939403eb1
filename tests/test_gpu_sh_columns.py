"""Inverse transforms whose workgroups take all column groups that fit, with one latitude tile per wave, against the
oracle."""
import numpy as np
import pytest

import synth
from oracle import sh as osh

pytestmark = pytest.mark.gpu

TOL = 5e-12   # as for the flat spectra of the other transform tests


# 4, 5, 6 and 8 groups of four columns to a workgroup
@pytest.mark.parametrize("T,nlat,nlon,B", [(300, 302, 1024, 8), (255, 256, 512, 20), (255, 256, 512, 23), (255, 256, 512, 32)])
def test_inverse_of_many_columns(T, nlat, nlon, B):
    import torch
    import paper_1812_03431_amd as rexi
    print(f"\n[gpu] inverse columns T={T} B={B}", flush=True)
    w = synth.Workload("sh", T=T, nlat=nlat, nlon=nlon, dt=3600.0, M=8, states=1)
    plan = rexi.plan_for(w, max_fields=B)
    rng = np.random.default_rng(T + B)
    spec = rng.standard_normal((B, plan.nspec)) + 1j * rng.standard_normal((B, plan.nspec))
    spec[:, :T + 1] = spec[:, :T + 1].real
    want = osh.synthesis(spec, T, nlat, nlon)
    got = plan.sh_inverse(torch.from_numpy(spec).to("cuda:0")).cpu().numpy()
    assert np.max(np.abs(got - want)) / np.max(np.abs(want)) < TOL
