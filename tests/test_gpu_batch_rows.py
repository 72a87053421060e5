"""A batch's fields bit for bit against the per-field launches where a
contiguous row of the coarse grid is too long for the batch's staging (4096
nodes) and there are too few rows for chunks: 4097 coarse nodes in fewer than
16 rows, and one row more and one level less, on white noise (neighbouring
separators of very different size, so that an eliminated separator rounds
differently from one taken by itself).
"""
import pytest
import torch

import paper_2007_04457_amd as mgr

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

SHAPES = [(8193,), (16385,), (17, 8193), (33, 8193), (5, 9, 8193), (4097,)]


@pytest.mark.parametrize("dt", [torch.float32, torch.float64], ids=["f32", "f64"])
def test_noise_equals_per_field(dt):
    shapes = SHAPES * 3
    gen = torch.Generator().manual_seed(71)
    xs = [torch.randn(s, dtype=torch.float64, generator=gen).to(dt).to(DEV) for s in shapes]
    plan = mgr.BatchPlan(shapes, dt)
    for persistent in (False, True):
        plan.set_mode(persistent)
        ys = plan.decompose(xs)
        plan.check()
        for x, y in zip(xs, ys):
            assert torch.equal(y, mgr.decompose(x)), (persistent, tuple(x.shape))
