"""Level steps on both sides of the lines between the single-workgroup tail
and launches of their own, against the CPU FP64 oracle in all four directions:
tables in the LDS or past it, dimensions of few and of many fibres, long and
short chains of taps, up to the default number of nodes; and that number as
the caller sets it, which holds for every grid alike.

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

SHAPES = [(17, 17, 33), (33, 17, 17), (65, 129), (129, 65), (33, 257), (257, 33), (9, 257), (9, 513), (513, 5), (17, 513),
          (5, 9, 129), (129, 9, 5), (3, 17, 129), (9, 17, 65), (513,), (257,), (65, 65), (33, 129)]


@pytest.mark.parametrize("dt", [torch.float32, torch.float64], ids=["f32", "f64"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_matches_oracle(shape, dt):
    for L in sorted({1, oracle.max_levels(shape)}):
        u, coords = synth.sinusoid_field(shape, 94, nonuniform=True)
        x = torch.from_numpy(u).to(dt)
        xd, xg = x.double().numpy(), x.to(DEV)
        scale = float(np.max(np.abs(xd)))
        for name in ("decompose", "recompose", "decompose_adjoint"):
            got = getattr(mgr, name)(xg, coords, L).double().cpu().numpy()
            want = getattr(oracle, name)(xd, coords, L)
            assert float(np.max(np.abs(got - want))) / scale <= TOL[dt], (name, L)
        got = mgr.recompose_adjoint(xg, coords, L).double().cpu().numpy()
        want = oracle.recompose_adjoint(xd, coords, L)
        # (its outputs grow from step to step)
        assert float(np.max(np.abs(got - want))) / max(scale, float(np.max(np.abs(want)))) <= TOL[dt], L


@pytest.mark.parametrize("shape", [(9, 513), (17, 17, 16 + 1), (65, 65)], ids=lambda s: "x".join(map(str, s)))
def test_number_of_nodes_is_the_callers(shape):
    """A single step joins the tail from exactly as many nodes on as it has,
    also where a dimension has few fibres."""
    n = int(np.prod(shape))
    x = torch.from_numpy(synth.sinusoid_field(shape, 95)[0]).to(torch.float32).to(DEV)
    mgr.decompose(x, None, 1)
    prev = mgr.mgr_set_tail_max_nodes(n)
    try:
        counts = []
        for limit in (n, n - 1):
            mgr.mgr_set_tail_max_nodes(limit)
            mgr.mgr_timing_enable("tail", 0)
            mgr.decompose(x, None, 1)
            counts.append(mgr.mgr_timing_read()[1])
            mgr.mgr_timing_disable()
        assert counts == [1, 0]
    finally:
        mgr.mgr_set_tail_max_nodes(prev)
