"""The per-stage kernels of general grids, which run planes of 2 GiB and more
and 4-D planes past the LDS, against the CPU FP64 oracle: at small sizes
through the test switch, in one to four dimensions and both types, and at the
sizes that reach them by themselves; and the line at 2 GiB.

Tolerances (max |gpu - oracle| / max |input|): 1e-12 in float64, 2e-5 in
float32, as for the other grids.
"""
import threading

import numpy as np
import pytest
import torch

import oracle
import paper_2007_04457_amd as mgr
from paper_2007_04457_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
TOL = {torch.float64: 1e-12, torch.float32: 2e-5}

SHAPES = [(4,), (100,), (1000,), (5000,), (4, 6), (10, 9), (130, 256), (3, 3000), (600, 50), (4, 4, 4), (7, 8, 9), (33, 20, 17),
          (40, 66, 65), (20, 3, 13), (1030, 6, 5), (3, 3, 3, 3), (6, 7, 12, 5), (5, 17, 9, 9), (12, 11, 10, 9)]


@pytest.fixture
def per_stage():
    prev = mgr.mgr_set_per_stage(True)
    yield
    mgr.mgr_set_per_stage(prev)


def check(shape, dt, coords, u, L):
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
    z = yr.to(DEV)
    mgr.mgr_recompose(z, z, coords, L)
    assert torch.equal(z, r), L


@pytest.mark.parametrize("dt", [torch.float32, torch.float64], ids=["f32", "f64"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_matches_oracle(shape, dt, per_stage):
    full = oracle.max_levels(shape)
    for nonuniform, L in ((True, -1), (False, full + 1), (True, min(1, full))):
        u, coords = synth.sinusoid_field(shape, 102, nonuniform=nonuniform)
        mgr.mgr_timing_enable("coef_decompose", 0)
        check(shape, dt, coords, u, L)
        n = mgr.mgr_timing_read()[1]
        mgr.mgr_timing_disable()
        steps = full if L < 0 else L
        assert n == (2 if steps > 0 else 0), L  # both decompositions by the per-stage coefficient kernel


@pytest.mark.parametrize("dt", [torch.float32, torch.float64], ids=["f32", "f64"])
def test_planes_past_the_lds(dt):
    shape = (3, 4, 200, 200)  # 244 KB of LDS in FP32
    u, coords = synth.sinusoid_field(shape, 103, nonuniform=True)
    check(shape, dt, coords, u, 1)


def test_switch_is_the_threads_own(per_stage):
    seen = []
    t = threading.Thread(target=lambda: seen.append(mgr.mgr_set_per_stage(False)))
    t.start()
    t.join()
    assert seen == [False] and mgr.mgr_set_per_stage(True) is True


def test_line_at_2_gib():
    """The largest plane that the fused kernels address and the smallest that
    they do not (FP64, 2^28 - 2^14 and 2^28 nodes): one column more or less
    changes nothing far from it, where a column's influence has decayed below
    rounding."""
    dt, keep = torch.float64, 16000
    gen = torch.Generator(device=DEV).manual_seed(104)
    wide = torch.randn((3, 16384, 16384), dtype=dt, device=DEV, generator=gen)
    y = mgr.decompose(wide, None, 1)
    r = mgr.recompose(y, None, 1)
    scale = float(wide.abs().max())
    assert float((r - wide).abs().max()) / scale <= 1e-11
    del r
    narrow = wide[:, :, :16383].contiguous()
    del wide
    z = mgr.decompose(narrow, None, 1)
    assert float((z[:, :, :keep] - y[:, :, :keep]).abs().max()) / scale <= 1e-12
    del y
    r = mgr.recompose(z, None, 1)
    assert float((r - narrow).abs().max()) / scale <= 1e-11
    del r, z, narrow
    torch.cuda.synchronize()
    mgr.mgr_finalize()
    torch.cuda.empty_cache()
