"""Class packing and the quantiser at the sizes where their work splits: rows
shorter and longer than a lane group (17, 33, 65 columns) and than a row piece
(2048), one dimension, few and many rows, every level count; quantisation of
packed arrays whose spans lie inside one class, cross class boundaries or end
early, at 16-byte aligned and unaligned addresses, with values that clamp.
All bit for bit against the CPU oracle.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2007_04457_amd as mgr

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

SHAPES = [(3, 3, 3), (9, 17, 17), (17, 9, 33), (5, 33, 65), (33, 65, 129), (3, 5, 2049), (2049, 9), (9, 4097), (65, 3),
          (3,), (33,), (8193,), (129, 5, 9)]


def values(n, dt, seed):
    return torch.from_numpy(np.random.default_rng(seed).normal(size=n)).to(dt)


@pytest.mark.parametrize("dt", [torch.float32, torch.float64], ids=["f32", "f64"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_pack_unpack(shape, dt):
    full = oracle.max_levels(shape)
    y = values(shape, dt, 81)
    for L in sorted({0, min(1, full), full, full + 1}):
        want = oracle.pack_classes(y.double().numpy(), L)
        p = mgr.pack_classes(y.to(DEV), L)
        assert np.array_equal(p.double().cpu().numpy(), want), L
        assert torch.equal(mgr.unpack_classes(p, shape, L).cpu(), y), L


@pytest.mark.parametrize("off", [0, 1, 3], ids=lambda o: f"off{o}")
@pytest.mark.parametrize("dt", [torch.float32, torch.float64], ids=["f32", "f64"])
@pytest.mark.parametrize("shape", [(3,), (33, 65), (33, 65, 129), (17, 129, 65)], ids=lambda s: "x".join(map(str, s)))
def test_quantize_packed(shape, dt, off):
    n = int(np.prod(shape))
    L = oracle.max_levels(shape)
    bins = np.array([0.3 * 0.7 ** c for c in range(L + 1)])
    p = values(n, dt, 82)
    p[0], p[n // 2], p[n - 1] = float("nan"), 1e30, float("-inf")
    buf = torch.zeros(n + 8, dtype=dt, device=DEV)
    buf[off:off + n] = p.to(DEV)
    cb = torch.full((n + 8,), 77, dtype=torch.int32, device=DEV)
    codes, clamped = mgr.quantize(buf[off:off + n], bins, shape, L, packed=True, codes=cb[off:off + n])
    want, wn = oracle.quantize(p.numpy(), bins, L, True, shape)
    assert np.array_equal(codes.cpu().numpy(), want.reshape(-1)) and int(clamped) == wn
    assert bool((cb[:off] == 77).all()) and bool((cb[off + n:] == 77).all())
    ob = torch.full((n + 8,), 5.0, dtype=dt, device=DEV)
    back = mgr.dequantize(codes, bins, dt, shape, L, packed=True, out=ob[off:off + n])
    assert np.array_equal(back.cpu().numpy(), oracle.dequantize(want, bins, p.numpy().dtype, L, True, shape).reshape(-1))
    assert bool((ob[:off] == 5.0).all()) and bool((ob[off + n:] == 5.0).all())
