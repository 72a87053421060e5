"""Any-length grids of 1 to 3 dimensions on the fused streaming kernels
against the CPU FP64 oracle, at the sizes where the phantom node before the
last node of an even-length level grid can go wrong: even and odd in every
combination, one node more or less than a tile's rows (16 fine rows) and
columns (60, 64, 124, 252), a last node that is the first row or column of a
tile, even lengths at deeper level grids, planes split into chunks, the
smallest sizes.

Tolerances (max |gpu - oracle| / max |input|): 1e-12 in float64, 2e-5 in
float32, as for the 2^k + 1 sizes.
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

SHAPES = [
    (4, 4, 4), (3, 4, 6), (6, 3, 4), (4, 6, 3), (7, 8, 9), (16, 16, 16), (17, 18, 62), (18, 17, 61), (34, 32, 64),
    (33, 34, 66), (5, 16, 124), (12, 48, 126), (40, 66, 65), (66, 33, 254), (20, 130, 70), (130, 6, 10),
    (18, 18, 17), (19, 19, 19), (21, 21, 21),
    (4, 4), (3, 6), (6, 3), (17, 252), (40, 254), (130, 256), (257, 258), (600, 50), (50, 600),
    (4,), (6,), (7,), (64,), (254,), (255,), (1030,), (5000,),
]


def sid(s):
    return "x".join(map(str, s))


def field(shape, seed, nonuniform, dtype):
    u, coords = synth.sinusoid_field(shape, seed, nonuniform=nonuniform)
    x = torch.from_numpy(u).to(dtype)
    return x, x.double().numpy(), coords


@pytest.mark.parametrize("dt", [torch.float32, torch.float64], ids=["f32", "f64"])
@pytest.mark.parametrize("shape", SHAPES, ids=sid)
def test_matches_oracle(shape, dt):
    full = oracle.max_levels(shape)
    for nonuniform, L in ((False, -1), (True, full + 1), (True, min(1, full))):
        x, xd, coords = field(shape, 51, nonuniform, dt)
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


@pytest.mark.parametrize("offset", [1, 7, 31])
def test_output_off_line_boundaries(offset):
    """The finest recomposition aligns its stores to the output's cache
    lines: outputs that start anywhere in a line give the same bits, and
    nothing outside them is written."""
    shape = (20, 34, 150)
    x = field(shape, 52, False, torch.float32)[0].to(DEV)
    y = mgr.decompose(x)
    want = mgr.recompose(y)
    n = x.numel()
    buf = torch.full((n + 256,), 7.0, dtype=torch.float32, device=DEV)
    out = buf[offset:offset + n].view(shape)
    mgr.mgr_recompose(y, out)
    assert torch.equal(out, want)
    assert bool((buf[:offset] == 7.0).all()) and bool((buf[offset + n:] == 7.0).all())


def test_captured_recomposition_replays():
    """Capture of a general recomposition keeps to the captured stream; every
    replay equals the eager result."""
    shape = (30, 44, 70)
    x = field(shape, 53, False, torch.float32)[0].to(DEV)
    y = mgr.decompose(x)
    want = mgr.recompose(y)
    out = torch.empty_like(x)
    g = torch.cuda.CUDAGraph()
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        with torch.cuda.graph(g, stream=st):
            mgr.mgr_recompose(y, out)
    for _ in range(3):
        out.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want)
        assert torch.equal(mgr.recompose(y), want)
