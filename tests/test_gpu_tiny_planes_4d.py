"""Four-dimensional grids of very many tiny planes on both sides of the line
between the plane kernels and the per-stage kernels, against the CPU FP64
oracle, in place and out of place.

Tolerances (max |gpu - oracle| / max |input|): 1e-12 in float64, 2e-5 in
float32, as for the other grids.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2007_04457_amd as mgr
from paper_2007_04457_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
TOL = {torch.float64: 1e-12, torch.float32: 2e-5}

# planes * (38 - nodes) (FP64: 58) on either side of 500000
SHAPES = [(150, 115, 3, 3), (106, 96, 3, 3), (106, 97, 3, 3), (200, 190, 5, 5), (131, 131, 4, 4), (240, 210, 6, 8), (8, 2200, 3, 4)]


@pytest.mark.parametrize("dt", [torch.float32, torch.float64], ids=["f32", "f64"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_matches_oracle(shape, dt):
    u, coords = synth.sinusoid_field(shape, 96, nonuniform=True)
    x = torch.from_numpy(u).to(dt)
    xd, xg = x.double().numpy(), x.to(DEV)
    y = mgr.decompose(xg, coords, 1)
    want = oracle.decompose(xd, coords, 1)
    assert float(np.max(np.abs(y.double().cpu().numpy() - want))) / float(np.max(np.abs(xd))) <= TOL[dt]
    yr = torch.from_numpy(want).to(dt)
    r = mgr.recompose(yr.to(DEV), coords, 1)
    wr = oracle.recompose(yr.double().numpy(), coords, 1)
    assert float(np.max(np.abs(r.double().cpu().numpy() - wr))) / float(yr.abs().max()) <= TOL[dt]
    z = xg.clone()
    mgr.mgr_decompose(z, z, coords, 1)
    assert torch.equal(z, y)
    z = yr.to(DEV)
    mgr.mgr_recompose(z, z, coords, 1)
    assert torch.equal(z, r)


@pytest.mark.parametrize("shape,launches", [((40, 50, 5, 5), 3), ((20, 20, 5, 5), 1)], ids=["planes-alone", "together"])
def test_timing_counts_launches_made(shape, launches):
    """Solve launches of the finest step: the planes' and one for each of dims 1
    and 0 where there are more planes than CUs; otherwise the planes are solved
    with their load vector and dims 1 and 0 in one launch."""
    x = torch.from_numpy(synth.sinusoid_field(shape, 101)[0]).to(DEV)
    mgr.decompose(x, None, 1)
    mgr.mgr_timing_enable("solve", 0)
    mgr.decompose(x, None, 1)
    n = mgr.mgr_timing_read()[1]
    mgr.mgr_timing_disable()
    assert n == launches
