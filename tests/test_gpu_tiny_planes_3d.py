"""Any-length 3-D grids of very many tiny planes on both sides of the line
between the fused kernels and the per-stage kernels, against the CPU FP64
oracle, in place and out of place.

Past the line the results are the per-stage kernels' bits.  Tolerances
(max |gpu - oracle| / max |input|): 1e-12 in float64, 2e-5 in float32, as for
the other grids.
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
EVEN = {torch.float64: 100, torch.float32: 70}

# planes * (even - nodes) on either side of 400000 a level step: FP64 4705 and
# 4706 planes, FP32 7272 and 7273 of 3 x 5 nodes; then more nodes, one and two steps
SHAPES = [(4705, 3, 5), (4706, 3, 5), (7272, 3, 5), (7273, 3, 5), (30000, 3, 4), (30001, 4, 3), (22000, 7, 9), (58000, 7, 9),
          (22000, 9, 11), (6000, 3, 33)]


@pytest.mark.parametrize("dt", [torch.float32, torch.float64], ids=["f32", "f64"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_matches_oracle(shape, dt):
    u, coords = synth.sinusoid_field(shape, 103, nonuniform=True)
    x = torch.from_numpy(u).to(dt)
    xd, xg = x.double().numpy(), x.to(DEV)
    nodes = shape[1] * shape[2]
    for L in range(1, oracle.max_levels(shape) + 1):
        stages = nodes < EVEN[dt] and shape[0] * (EVEN[dt] - nodes) > 400000 * L
        y = mgr.decompose(xg, coords, L)
        want = oracle.decompose(xd, coords, L)
        assert float(np.max(np.abs(y.double().cpu().numpy() - want))) / float(np.max(np.abs(xd))) <= TOL[dt], L
        yr = torch.from_numpy(want).to(dt)
        r = mgr.recompose(yr.to(DEV), coords, L)
        wr = oracle.recompose(yr.double().numpy(), coords, L)
        assert float(np.max(np.abs(r.double().cpu().numpy() - wr))) / float(yr.abs().max()) <= TOL[dt], L
        z = xg.clone()
        mgr.mgr_decompose(z, z, coords, L)
        assert torch.equal(z, y), L
        z = yr.to(DEV)
        mgr.mgr_recompose(z, z, coords, L)
        assert torch.equal(z, r), L
        if stages:
            mgr.mgr_set_per_stage(True)
            try:
                assert torch.equal(mgr.decompose(xg, coords, L), y), L
                assert torch.equal(mgr.recompose(yr.to(DEV), coords, L), r), L
            finally:
                mgr.mgr_set_per_stage(False)
