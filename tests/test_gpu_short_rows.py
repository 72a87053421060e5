"""Any-length 3-D grids of short rows on both sides of the line between narrow
tiles (up to 30 coarse columns) and wide ones, against the CPU FP64 oracle, in
place and out of place: rows of 29 to 32 coarse nodes, one and several tiles
of rows, planes in one chunk and in many.

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

SHAPES = [(20, 40, 56), (20, 40, 57), (20, 40, 58), (21, 17, 59), (20, 40, 60), (12, 33, 61), (12, 34, 62), (3000, 6, 7),
          (1030, 60, 6), (1500, 4, 3), (40, 130, 59)]


@pytest.mark.parametrize("dt", [torch.float32, torch.float64], ids=["f32", "f64"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_matches_oracle(shape, dt):
    for L in sorted({1, oracle.max_levels(shape)}):
        if L < 1:
            continue
        u, coords = synth.sinusoid_field(shape, 99, nonuniform=True)
        x = torch.from_numpy(u).to(dt)
        xd, xg = x.double().numpy(), x.to(DEV)
        y = mgr.decompose(xg, coords, L)
        want = oracle.decompose(xd, coords, L)
        assert float(np.max(np.abs(y.double().cpu().numpy() - want))) / float(np.max(np.abs(xd))) <= TOL[dt], L
        yr = torch.from_numpy(want).to(dt)
        r = mgr.recompose(yr.to(DEV), coords, L)
        wr = oracle.recompose(yr.double().numpy(), coords, L)
        assert float(np.max(np.abs(r.double().cpu().numpy() - wr))) / float(yr.abs().max()) <= TOL[dt], L
        z = xg.clone()  # in place: the same bits
        mgr.mgr_decompose(z, z, coords, L)
        assert torch.equal(z, y), L
