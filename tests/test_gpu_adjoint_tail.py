"""Adjoints of the decomposition and the recomposition against the CPU FP64
oracle where they change form: level grids that one workgroup takes from the
first step on, and from a later one; one, two and three active dimensions of
few and of many fibres; long first dimensions (the first solve reads another
array, in one launch and in chunks); truncated level counts; in place.

Tolerances as for the other adjoint tests: 1e-12 (float64), 2e-5 (float32),
of the input's scale, and for the recomposition of the largest value that any
of its steps handles.
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

SHAPES = [(3,), (5,), (9,), (33,), (257,), (513,), (1025,), (3, 3), (3, 5), (5, 3), (9, 33), (33, 9), (65, 65), (3, 513),
          (513, 3), (257, 17), (2049, 5), (5, 2049), (3, 3, 3), (5, 3, 9), (3, 65, 3), (9, 9, 9), (17, 17, 17),
          (5, 129, 5), (65, 5, 9), (9, 17, 33), (33, 33, 33), (129, 9, 17), (17, 65, 129), (1025, 5, 9), (17, 17, 33), (129, 65),
          (257, 33)]


@pytest.mark.parametrize("dt", [torch.float32, torch.float64], ids=["f32", "f64"])
@pytest.mark.parametrize("shape", SHAPES, ids=["x".join(map(str, s)) for s in SHAPES])
def test_matches_oracle(shape, dt):
    full = oracle.max_levels(shape)
    for nonuniform, L in ((False, full), (True, full), (True, max(1, full - 1))):
        g, coords = synth.sinusoid_field(shape, 71, nonuniform=nonuniform)
        g = torch.from_numpy(g).to(dt)
        gd = g.double().numpy()
        gg = g.to(DEV)
        a = mgr.decompose_adjoint(gg, coords, L)
        want = oracle.decompose_adjoint(gd, coords, L)
        assert np.max(np.abs(a.double().cpu().numpy() - want)) / np.max(np.abs(gd)) <= TOL[dt], (nonuniform, L)
        r = mgr.recompose_adjoint(gg, coords, L)
        scale = np.max(np.abs(gd))
        for k in range(L + 1):
            G = oracle.recompose_adjoint(gd, coords, k)[tuple(slice(None, None, 2 ** k) for _ in shape)]
            scale = max(scale, np.max(np.abs(G)))
        want = oracle.recompose_adjoint(gd, coords, L)
        assert np.max(np.abs(r.double().cpu().numpy() - want)) / scale <= TOL[dt], (nonuniform, L)
        for fn, out in ((mgr.mgr_decompose_adjoint, a), (mgr.mgr_recompose_adjoint, r)):  # in place: the same bits
            z = gg.clone()
            fn(z, z, coords, L)
            assert torch.equal(z, out), (nonuniform, L)
