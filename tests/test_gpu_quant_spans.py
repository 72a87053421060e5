"""Quantisation of packed arrays on both sides of the line between one and four
accesses in flight per lane, bit for bit against the CPU oracle: aligned and
unaligned addresses, clamped values in the first, an inner and the last span,
many classes in the first span.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2007_04457_amd as mgr

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

CASES = [((65, 513, 1025), torch.float32, 0), ((4097, 4097), torch.float64, 0), ((4097, 2049), torch.float64, 0), ((2049, 2049), torch.float64, 0),
         ((2049, 2049), torch.float32, 1), ((2**20 + 1,), torch.float32, 0), ((2**20 + 1,), torch.float64, 1)]


@pytest.mark.parametrize("case", CASES, ids=[f"{'x'.join(map(str, c[0]))}-{str(c[1])[6:]}-off{c[2]}" for c in CASES])
def test_quantize_packed(case):
    shape, dt, off = case
    n, L = int(np.prod(shape)), oracle.max_levels(shape)
    bins = np.array([0.3 * 0.7 ** c for c in range(L + 1)])
    p = torch.from_numpy(np.random.default_rng(98).normal(size=n)).to(dt)
    p[0], p[n // 2], p[n // 2 + 1], p[n - 1] = float("nan"), 1e30, float("-inf"), float("inf")
    buf = torch.zeros(n + 4, dtype=dt, device=DEV)
    buf[off:off + n] = p.to(DEV)
    codes, clamped = mgr.quantize(buf[off:off + n], bins, shape, L, packed=True)
    want, wn = oracle.quantize(p.numpy(), bins, L, True, shape)
    assert np.array_equal(codes.cpu().numpy().reshape(-1), want.reshape(-1)) and int(clamped) == wn
    back = mgr.dequantize(codes, bins, dt, shape, L, packed=True)
    assert np.array_equal(back.cpu().numpy().reshape(-1), oracle.dequantize(want, bins, p.numpy().dtype, L, True, shape).reshape(-1))
