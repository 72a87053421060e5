"""Class packing on both sides of the line between a wave per row piece and a
thread per node: row pieces (2304 columns) that split rows of three active
dimensions, the shortest rows and the fewest pieces that go by rows, one
less of each, one dimension; bit for bit against the CPU oracle, both ways.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2007_04457_amd as mgr

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# (rows, columns): rows of two pieces; 4096 pieces of over 192 columns and 65536 of 129 are where rows begin
SHAPES = [(5, 9, 4097), (9, 257, 4097), (257, 9, 4097), (4097, 257), (2049, 257), (4097, 129), (257, 257, 129),
          (129, 257, 129), (513, 9, 257), (16385,), (2**18 + 1,)]


@pytest.mark.parametrize("dt", [torch.float32, torch.float64], ids=["f32", "f64"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_pack_unpack(shape, dt):
    full = oracle.max_levels(shape)
    y = torch.from_numpy(np.random.default_rng(97).normal(size=shape)).to(dt)
    for L in sorted({1, full, full + 1}):
        p = mgr.pack_classes(y.to(DEV), L)
        assert np.array_equal(p.double().cpu().numpy(), oracle.pack_classes(y.double().numpy(), L)), L
        assert torch.equal(mgr.unpack_classes(p, shape, L).cpu(), y), L
