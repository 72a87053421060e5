"""Four-dimensional grids by planes of the last two dimensions against the CPU
FP64 oracle: even and odd lengths in every dimension, planes of one wave and
of several, long last dimensions (chunked solves), planes above 64 KB of LDS,
a plane too large for LDS (a thread per node), more planes than CUs, each
number of levels.

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

SHAPES = [(3, 3, 3, 3), (4, 3, 4, 3), (3, 4, 3, 4), (4, 4, 4, 4), (5, 6, 7, 8), (8, 7, 6, 5), (9, 10, 12, 11),
          (10, 9, 11, 12), (3, 20, 4, 33), (17, 4, 40, 5), (6, 5, 8, 16), (5, 6, 3, 700), (4, 5, 90, 91),
          (3, 4, 150, 140), (33, 34, 5, 6)]


@pytest.mark.parametrize("dt", [torch.float32, torch.float64], ids=["f32", "f64"])
@pytest.mark.parametrize("shape", SHAPES, ids=["x".join(map(str, s)) for s in SHAPES])
def test_matches_oracle(shape, dt):
    full = oracle.max_levels(shape)
    for nonuniform, L in ((True, -1), (False, full + 1), (True, 1)):
        u, coords = synth.sinusoid_field(shape, 61, nonuniform=nonuniform)
        x = torch.from_numpy(u).to(dt)
        xd = x.double().numpy()
        scale = float(np.max(np.abs(xd)))
        xg = x.to(DEV)
        y = mgr.decompose(xg, coords, L)
        want = oracle.decompose(xd, coords, L)
        assert float(np.max(np.abs(y.double().cpu().numpy() - want))) / scale <= TOL[dt], (nonuniform, L)
        yr = torch.from_numpy(want).to(dt)
        r = mgr.recompose(yr.to(DEV), coords, L)
        wr = oracle.recompose(yr.double().numpy(), coords, L)
        assert float(np.max(np.abs(r.double().cpu().numpy() - wr))) / float(yr.abs().max()) <= TOL[dt], (nonuniform, L)
        z = xg.clone()  # in place: the same bits
        mgr.mgr_decompose(z, z, coords, L)
        assert torch.equal(z, y), (nonuniform, L)
        z2 = y.clone()
        mgr.mgr_recompose(z2, z2, coords, L)
        assert torch.equal(z2, mgr.recompose(y, coords, L)), (nonuniform, L)
