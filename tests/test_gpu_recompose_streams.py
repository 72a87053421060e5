"""Recompositions by what runs beside the caller's stream: nothing (one
streamed level step and no tail), the tail alone, the finest correction alone
(no tail), both; 2^k + 1 and any-length grids, below and above the size up to
which the finest correction shares launches, against the CPU FP64 oracle,
eager and replayed from a capture.

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

# shape, dtype, level steps, tail
CASES = [((1000,), torch.float32, 1, True), ((4777,), torch.float64, 1, True), ((300, 70), torch.float64, 1, True),
         ((65, 65, 65), torch.float32, 1, True), ((129, 257, 129), torch.float64, 1, True),
         ((129, 257, 129), torch.float64, 2, False), ((120, 250, 100), torch.float64, 2, False),
         ((65, 33, 129), torch.float32, 2, False), ((4777,), torch.float32, 3, False),
         ((129, 257, 129), torch.float64, -1, True), ((120, 250, 100), torch.float64, -1, True),
         ((17, 4097), torch.float32, -1, True)]


@pytest.mark.parametrize("case", CASES, ids=[f"{'x'.join(map(str, c[0]))}-L{c[2]}-{'tail' if c[3] else 'notail'}"
                                             for c in CASES])
def test_streams(case):
    shape, dt, L, tail = case
    prev = mgr.mgr_set_tail_max_nodes(0) if not tail else None
    try:
        u, _ = synth.sinusoid_field(shape, 91)
        y = torch.from_numpy(u).to(dt)
        want = oracle.recompose(y.double().numpy(), None, L)
        yg = y.to(DEV)
        mgr.mgr_prepare(dt, shape, None, L)
        r = mgr.recompose(yg, None, L)
        assert float(np.max(np.abs(r.double().cpu().numpy() - want))) / float(y.abs().max()) <= TOL[dt]
        z = yg.clone()  # in place: the same bits
        mgr.mgr_recompose(z, z, None, L)
        assert torch.equal(z, r)
        out = torch.empty_like(yg)
        g = torch.cuda.CUDAGraph()
        st = torch.cuda.Stream()
        st.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(st):
            with torch.cuda.graph(g, stream=st):
                mgr.mgr_recompose(yg, out, None, L)
        for _ in range(3):
            out.zero_()
            g.replay()
            torch.cuda.synchronize()
            assert torch.equal(out, r)
            assert torch.equal(mgr.recompose(yg, None, L), r)
    finally:
        if prev is not None:
            mgr.mgr_set_tail_max_nodes(prev)
