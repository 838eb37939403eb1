"""The Legendre kernels at the edges of their segments, parts, runs, latitude tiles
and column groups, on flat spectra (every degree of every order counts alike),
against the oracle."""
import numpy as np
import pytest

import synth
from oracle import sh as osh

pytestmark = pytest.mark.gpu

# A recurrence of r degrees from exact values is off by at most about r^2 ulp (32
# degrees: 2.3e-13); twenty times that leaves room for the sums over degrees or
# latitudes and for the oracle's own recurrence.
TOL = 5e-12


# 128 degrees to an inverse segment (four parts of up to 32), 32 to a forward run and
# two runs to a workgroup; 16 latitudes to a tile, two tiles per wave from 1024
# workgroups on (T255 with 512 northern latitudes, not T254); 32 columns (16 fields)
# to a launch
@pytest.mark.parametrize("T,nlat,nlon,B", [(31, 32, 64, 16), (32, 34, 64, 2), (64, 66, 128, 3), (127, 128, 256, 1),
                                           (128, 130, 256, 4), (129, 132, 512, 5), (167, 260, 512, 7),
                                           (255, 1024, 512, 3), (254, 1024, 512, 17), (200, 514, 512, 6)])
def test_flat_spectra_match_oracle(T, nlat, nlon, B):
    import torch
    import paper_1812_03431_amd as rexi
    print(f"\n[gpu] sh tiles T={T} nlat={nlat} nlon={nlon} B={B}", flush=True)
    w = synth.Workload("sh", T=T, nlat=nlat, nlon=nlon, dt=3600.0, M=8, states=1)
    plan = rexi.plan_for(w, max_fields=B)
    rng = np.random.default_rng(T * 1000 + B)
    spec = rng.standard_normal((B, plan.nspec)) + 1j * rng.standard_normal((B, plan.nspec))
    spec[:, :T + 1] = spec[:, :T + 1].real
    want = osh.synthesis(spec, T, nlat, nlon)
    got = plan.sh_inverse(torch.from_numpy(spec).to("cuda:0")).cpu().numpy()
    err = np.max(np.abs(got - want)) / np.max(np.abs(want))
    assert err < TOL, f"sh_inverse rel max err {err}"
    grid = rng.standard_normal((B, nlat, nlon))
    want = osh.analysis(grid, T)
    got = plan.sh_forward(torch.from_numpy(grid).to("cuda:0")).cpu().numpy()
    err = np.max(np.abs(got - want)) / np.max(np.abs(want))
    assert err < TOL, f"sh_forward rel max err {err}"


# every FFT length (4 .. 4096: one to four register passes, several FFTs per wave up
# to one on eight waves), orders on both sides of nlon / 2 (where bins alias), and
# field counts that leave a group of FFTs incomplete
@pytest.mark.parametrize("bits", range(2, 13))
@pytest.mark.parametrize("aliased", [False, True])
def test_fft_lengths_match_oracle(bits, aliased):
    import torch
    import paper_1812_03431_amd as rexi
    nlon = 1 << bits
    T = min(nlon - 1 if aliased else nlon // 2 - 1, 40)
    nlat, B = 2 * ((T + 2) // 2) + 2, 3
    print(f"\n[gpu] fft nlon={nlon} T={T} nlat={nlat} B={B}", flush=True)
    w = synth.Workload("sh", T=T, nlat=nlat, nlon=nlon, dt=3600.0, M=8, states=1)
    plan = rexi.plan_for(w, max_fields=B)
    rng = np.random.default_rng(bits)
    spec = rng.standard_normal((B, plan.nspec)) + 1j * rng.standard_normal((B, plan.nspec))
    spec[:, :T + 1] = spec[:, :T + 1].real
    want = osh.synthesis(spec, T, nlat, nlon)
    got = plan.sh_inverse(torch.from_numpy(spec).to("cuda:0")).cpu().numpy()
    assert np.max(np.abs(got - want)) / np.max(np.abs(want)) < TOL
    grid = rng.standard_normal((B, nlat, nlon))
    want = osh.analysis(grid, T)
    got = plan.sh_forward(torch.from_numpy(grid).to("cuda:0")).cpu().numpy()
    assert np.max(np.abs(got - want)) / np.max(np.abs(want)) < TOL
