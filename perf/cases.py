"""Timed workloads of the refactoring library, over the range a program uses it on.

A case is a dict of plain values; `prepare` makes what a program holds before
the call (a field on the GPU, output buffers, the prepared problem), `run` is
one pass through the public entry points, `work` the bytes and operations the
pass cannot do without, and `exact` the same outputs in 64 bits from plain
torch operations that share nothing with the library.

Kinds of pass:
  dec     decompose one field
  rec     recompose one refactored field
  step    decompose, then recompose (a write followed by a read back)
  grad    the decomposition as a layer: forward, then backward
  gradrec the recomposition as a layer: forward, then backward
  batch   decompose many independent fields together through a plan
  save    class-pack a refactored field and quantise it to integer codes
  load    dequantise packed codes and recompose them, wholly (drop = 0) or to
          the grid `drop` levels coarser (a preview)
"""
import random

import numpy as np
import torch

import paper_2007_04457_amd as mgr

DEV = "cuda"
DTYPE = {"f32": torch.float32, "f64": torch.float64}


def _case(kind, shape, dtype="f32", nonuniform=False, levels=-1, drop=0, fields=0):
    return {"kind": kind, "shape": "x".join(str(n) for n in shape), "dtype": dtype, "nonuniform": nonuniform,
            "levels": levels, "drop": drop, "fields": fields}


def _named(name, *args, **kw):
    return dict(_case(*args, **kw), name=name)


def listed():
    return [
        # one block of a block-structured code, refactored by itself: launches and latency are all of it
        _named("dec_33_f32", "dec", (33, 33, 33)),
        # a small double-precision block read back
        _named("rec_65_f64", "rec", (65, 65, 65), "f64"),
        # the headline workload: a snapshot of a three-dimensional simulation, written and read back
        _named("step_513_f32", "step", (513, 513, 513)),
        # the same in double precision
        _named("step_513_f64", "step", (513, 513, 513), "f64"),
        # a large two-dimensional field on a stretched mesh
        _named("step_8193x8193_f64", "step", (8193, 8193), "f64", True),
        # a field whose sizes are what the simulation chose, not 2^k + 1
        _named("step_500_f32", "step", (500, 500, 500)),
        # space and time, or space and a parameter, on a stretched four-dimensional mesh
        _named("step_4d_f64", "step", (40, 50, 60, 70), "f64", True),
        # a loss on the coefficients: the decomposition in a training step
        _named("grad_257_f32", "grad", (257, 257, 257)),
        # the recomposition in a training step, with uneven sizes on a stretched mesh
        _named("gradrec_129x65x257_f64", "gradrec", (129, 65, 257), "f64", True),
        # many partitions and variables of one run, refactored together
        _named("batch_60_f32", "batch", (0,), fields=60),
        # the writing half of the lossy path: classes laid out one after the other, then quantised
        _named("save_513_f32", "save", (513, 513, 513)),
        # the reading half: a preview one level below full resolution
        _named("load_513_f32", "load", (513, 513, 513), drop=1),
    ]


# The number of nodes a drawn case may have at most (513^3).
MOST = 513 ** 3


def _dyadic(rng, nd, kmin, kmax, most=MOST):
    while True:
        shape = tuple(2 ** rng.randint(kmin, kmax) + 1 for _ in range(nd))
        if _count(shape) <= most:
            return shape


def _any_size(rng, nd, lo, hi, most):
    while True:
        shape = tuple(int(round(lo * (hi / lo) ** rng.random())) for _ in range(nd))
        if _count(shape) <= most:
            return shape


def draw(rng):
    kind = rng.choice(["dec", "rec", "step", "step", "general", "general", "grad", "gradrec", "batch", "save", "load"])
    dtype = rng.choice(["f32", "f32", "f64"])
    nonuniform = rng.random() < 0.4
    if kind == "general":  # any sizes, one to four dimensions
        nd = rng.choice([1, 2, 3, 3, 3, 4])
        lo, hi = {1: (100, 1000000), 2: (30, 6000), 3: (12, 500), 4: (6, 90)}[nd]
        shape = _any_size(rng, nd, lo, hi, 30000000)
        if nd == 1:
            nonuniform = False
        return _case(rng.choice(["dec", "rec", "step"]), shape, dtype, nonuniform)
    if kind == "batch":
        return _case("batch", (0,), dtype, fields=int(round(4 * 15 ** rng.random())))
    if kind in ("grad", "gradrec"):
        nd = rng.choice([2, 3, 3])
        return _case(kind, _dyadic(rng, nd, *{2: (5, 11), 3: (4, 8)}[nd], most=257 ** 3), dtype, nonuniform)
    if kind in ("save", "load"):
        nd = rng.choice([2, 3, 3])
        shape = _dyadic(rng, nd, *{2: (6, 13), 3: (4, 9)}[nd])
        return _case(kind, shape, dtype, drop=rng.randint(0, 2) if kind == "load" else 0)
    nd = rng.choice([1, 2, 2, 3, 3, 3, 3])
    shape = _dyadic(rng, nd, *{1: (9, 20), 2: (5, 13), 3: (4, 9)}[nd])
    if nd == 1:
        nonuniform = False
    levels = rng.choice([-1, -1, -1, 3])
    return _case(kind, shape, dtype, nonuniform, levels)


# ---- sizes ------------------------------------------------------------------

def _count(shape):
    n = 1
    for m in shape:
        n *= m
    return n


def _shape(case):
    return tuple(int(n) for n in case["shape"].split("x"))


def _full_levels(shape):
    return min((n - 2).bit_length() for n in shape) - 1


def _levels(case):
    return _full_levels(_shape(case)) if case["levels"] < 0 else case["levels"]


def _coarser(shape, steps):
    return tuple(((n - 2) >> steps) + 2 for n in shape)


def _batch_shapes(case):
    """Five three-dimensional partitions (33 to 257 nodes a side) to each large plane."""
    rng = random.Random(1000 + case["fields"])
    return [tuple(2 ** rng.randint(9, 12) + 1 for _ in range(2)) if f % 6 == 5 else
            tuple(2 ** rng.randint(5, 8) + 1 for _ in range(3)) for f in range(case["fields"])]


def _coords(case):
    """The mesh belongs to the case: a run refactors many fields on one mesh."""
    if not case["nonuniform"]:
        return None
    rng = random.Random(77)
    out = []
    for n in _shape(case):
        x = [0.0]
        for _ in range(n - 1):
            x.append(x[-1] + rng.uniform(0.5, 1.5))
        out.append([v / x[-1] for v in x])
    return [np.asarray(x, dtype=np.float64) for x in out]


# ---- inputs -----------------------------------------------------------------

def _field(shape, dtype, seed):
    """Eight plane waves and a little noise: what a simulation's snapshot is like."""
    gen = torch.Generator(device=DEV).manual_seed(seed)
    rng = random.Random(seed)
    nd = len(shape)
    out = torch.randn(shape, generator=gen, device=DEV, dtype=torch.float32).to(dtype).mul_(1e-3)
    axes = [torch.linspace(0, 6.283185307179586, n, device=DEV, dtype=torch.float64) for n in shape]
    for _ in range(8):
        amp, phase = rng.uniform(0.1, 1.0), rng.uniform(0.0, 6.28)
        arg = torch.full((1,) * (nd - 1), phase, device=DEV, dtype=torch.float64)
        for d in range(nd - 1):
            arg = arg + rng.randint(1, 6) * axes[d].reshape([-1 if e == d else 1 for e in range(nd - 1)])
        last = rng.randint(1, 6) * axes[-1]
        out.add_((arg.sin() * amp).to(dtype)[..., None] * last.cos().to(dtype))
        out.add_((arg.cos() * amp).to(dtype)[..., None] * last.sin().to(dtype))
    return out


def _classes(shape, levels):
    """The class of each node (0: the coarsest values, `levels`: the finest coefficients)."""
    cls = torch.zeros(shape, device=DEV, dtype=torch.int8)
    for c in range(1, levels + 1):  # a node leaves class < c where some index is off the grid of class c - 1
        step = 1 << (levels - c + 1)
        for d, n in enumerate(shape):
            i = torch.arange(n, device=DEV)
            off = ((i % step != 0) & (i != n - 1)).reshape([-1 if e == d else 1 for e in range(len(shape))])
            cls = torch.where(off & (cls < c), torch.full_like(cls, c), cls)
    return cls


def _refactored(shape, dtype, levels, seed):
    """Coarsest values of order one, and coefficients that shrink by four from class to class, as a smooth field's do."""
    gen = torch.Generator(device=DEV).manual_seed(seed)
    size = torch.tensor([1.0] + [4.0 ** -c for c in range(1, levels + 1)], device=DEV, dtype=torch.float32)
    y = torch.randn(shape, generator=gen, device=DEV, dtype=torch.float32)
    return y.mul_(size[_classes(shape, levels).to(torch.int32)]).to(dtype)


def _bins(shape, levels):
    return mgr.quant_bins(len(shape), levels, 1e-4)


def _codes(shape, dtype, levels, seed):
    """Class-packed integer codes, of the sizes that quantised coefficients have."""
    gen = torch.Generator(device=DEV).manual_seed(seed)
    bins = _bins(shape, levels)
    grids = [_coarser(shape, levels - c) for c in range(levels + 1)]
    ends = [_count(g) for g in grids]
    codes = torch.empty(_count(shape), device=DEV, dtype=torch.int32)
    for c in range(levels + 1):
        lo = ends[c - 1] if c else 0
        v = torch.randn(ends[c] - lo, generator=gen, device=DEV, dtype=torch.float32)
        codes[lo:ends[c]] = (v * (4.0 ** -c / float(bins[c]))).round_().to(torch.int32)
    return codes


def prepare(case, seed):
    kind, dtype = case["kind"], DTYPE[case["dtype"]]
    if kind == "batch":
        shapes = _batch_shapes(case)
        xs = [_field(s, dtype, seed * 1000 + f) for f, s in enumerate(shapes)]
        return {"kind": kind, "x": xs, "y": [torch.empty_like(x) for x in xs], "plan": mgr.BatchPlan(shapes, dtype)}
    shape, levels, coords = _shape(case), _levels(case), _coords(case)
    s = {"kind": kind, "shape": shape, "levels": case["levels"], "coords": coords, "dtype": dtype}
    if kind in ("dec", "step", "grad"):
        s["x"] = _field(shape, dtype, seed)
    elif kind in ("rec", "gradrec", "save"):
        s["x"] = _refactored(shape, dtype, levels, seed)
    if kind in ("dec", "rec"):
        s["out"] = torch.empty_like(s["x"])
    elif kind == "step":
        s["y"], s["out"] = torch.empty_like(s["x"]), torch.empty_like(s["x"])
    elif kind in ("grad", "gradrec"):
        s["x"].requires_grad_(True)
        s["g"] = _field(shape, dtype, seed + 500009)
    elif kind == "save":
        s["bins"] = _bins(shape, levels)
        s["packed"] = torch.empty(_count(shape), device=DEV, dtype=dtype)
        s["codes"] = torch.empty(_count(shape), device=DEV, dtype=torch.int32)
    elif kind == "load":
        s["bins"] = _bins(shape, levels)
        s["codes"] = _codes(shape, dtype, levels, seed)
        s["packed"] = torch.empty(_count(shape), device=DEV, dtype=dtype)
        s["level"] = max(0, levels - case["drop"])
        s["out"] = torch.empty(_coarser(shape, levels - s["level"]), device=DEV, dtype=dtype)
    if kind == "load":
        mgr.mgr_prepare(dtype, tuple(s["out"].shape), None, s["level"])
    elif kind != "save":
        mgr.mgr_prepare(dtype, shape, coords, case["levels"])
    return s


# ---- the pass ---------------------------------------------------------------

def run(s):
    kind = s["kind"]
    if kind == "batch":
        return s["plan"].decompose(s["x"], s["y"])
    if kind == "dec":
        return mgr.decompose(s["x"], s["coords"], s["levels"], out=s["out"])
    if kind == "rec":
        return mgr.recompose(s["x"], s["coords"], s["levels"], out=s["out"])
    if kind == "step":
        y = mgr.decompose(s["x"], s["coords"], s["levels"], out=s["y"])
        return y, mgr.recompose(y, s["coords"], s["levels"], out=s["out"])
    if kind in ("grad", "gradrec"):
        layer = mgr.Decompose if kind == "grad" else mgr.Recompose
        y = layer.apply(s["x"], s["coords"], s["levels"])
        g, = torch.autograd.grad(y, s["x"], s["g"])
        return y.detach(), g
    if kind == "save":
        p = mgr.pack_classes(s["x"], s["levels"], out=s["packed"])
        codes, clamped = mgr.quantize(p, s["bins"], s["shape"], s["levels"], packed=True, codes=s["codes"])
        return codes, clamped
    v = mgr.dequantize(s["codes"], s["bins"], s["dtype"], s["shape"], s["levels"], packed=True, out=s["packed"])
    return mgr.recompose_level(v, s["level"], s["shape"], None, s["levels"], packed=True, out=s["out"])


def work(case):
    """Each input read once and each output written once; about 20 operations a node for a pass over all levels."""
    b = 4 if case["dtype"] == "f32" else 8
    kind = case["kind"]
    if kind == "batch":
        n = sum(_count(s) for s in _batch_shapes(case))
        return {"bytes": 2 * n * b, "flops": 20 * n}
    n = _count(_shape(case))
    if kind in ("step", "grad", "gradrec"):
        return {"bytes": 4 * n * b, "flops": 40 * n}
    if kind == "save":
        return {"bytes": n * (b + 4), "flops": 2 * n}
    if kind == "load":
        m = _count(_coarser(_shape(case), min(_levels(case), case["drop"])))
        return {"bytes": m * (b + 4), "flops": 21 * m}
    return {"bytes": 2 * n * b, "flops": 20 * n}


# ---- the same in 64 bits, from plain torch operations -----------------------
#
# A level grid of m nodes along a dimension keeps its even positions and its
# last node; C = (I - P) u at the others, f = (P^T M) C along every dimension,
# M_c z = f along every dimension, and z is added to the kept values.

def _along(v, nd, d):
    return v.reshape([-1 if e == d else 1 for e in range(nd)])


class _Axis:
    """One dimension of one level grid: positions x, kept positions, interpolation and mass matrices."""

    def __init__(self, x, nd, d):
        m, self.d = x.numel(), d
        keep = torch.cat([torch.arange(0, m - 1, 2, device=DEV), torch.tensor([m - 1], device=DEV)])
        self.keep, self.xc = keep, x[keep]
        j = torch.arange(m, device=DEV)
        fine = (j % 2 == 1) & (j != m - 1)
        lo = torch.where(j == m - 1, torch.tensor(keep.numel() - 1, device=DEV), j // 2)
        self.lo, self.hi = lo, torch.where(fine, lo + 1, lo)
        up, dn = (j + 1).clamp(max=m - 1), (j - 1).clamp(min=0)
        a = torch.where(fine, (x - x[dn]) / (x[up] - x[dn]), torch.zeros_like(x))
        self.a = _along(a, nd, d)
        self.left, self.right = dn[keep], up[keep]
        self.wl = _along(torch.where(fine[self.left], a[self.left], torch.zeros_like(self.xc)), nd, d)
        self.wr = _along(torch.where(fine[self.right], 1 - a[self.right], torch.zeros_like(self.xc)), nd, d)
        self.hl, self.hr, self.diag = (_along(v, nd, d) for v in self._mass(x))
        self.dn, self.up, self.nd = dn, up, nd

    @staticmethod
    def _mass(x):
        h, z = x[1:] - x[:-1], torch.zeros(1, device=DEV, dtype=torch.float64)
        hl, hr = torch.cat([z, h]), torch.cat([h, z])
        return hl, hr, 2 * (hl + hr)

    def prolong(self, z):
        zl, zr = z.index_select(self.d, self.lo), z.index_select(self.d, self.hi)
        return zl + self.a * (zr - zl)

    def mass_restrict(self, c):
        w = self.diag * c + self.hl * c.index_select(self.d, self.dn) + self.hr * c.index_select(self.d, self.up)
        return (w.index_select(self.d, self.keep) + self.wl * w.index_select(self.d, self.left)
                + self.wr * w.index_select(self.d, self.right))

    def solve(self, f):
        """Parallel cyclic reduction: each step doubles the distance of the coupling, until there is none left."""
        lo, up, dg = self._mass(self.xc)
        n, s = self.xc.numel(), 1
        while s < n:
            i = torch.arange(n, device=DEV)
            dn, us = (i - s).clamp(min=0), (i + s).clamp(max=n - 1)
            k = torch.where(i >= s, -lo / dg[dn], torch.zeros_like(lo))
            g = torch.where(i + s < n, -up / dg[us], torch.zeros_like(lo))
            if float(torch.maximum(k.abs().max(), g.abs().max())) < 1e-20:
                break
            f = f + _along(k, self.nd, self.d) * f.index_select(self.d, dn) \
                + _along(g, self.nd, self.d) * f.index_select(self.d, us)
            dg = dg + k * up[dn] + g * lo[us]
            lo, up = k * lo[dn], g * up[us]
            s *= 2
        return f / _along(dg, self.nd, self.d)


def _axes(shape, coords):
    xs = [torch.arange(n, device=DEV, dtype=torch.float64) if coords is None else
          torch.as_tensor(coords[d], device=DEV, dtype=torch.float64) for d, n in enumerate(shape)]
    return [_Axis(x / (x[-1] - x[0]) * (x.numel() - 1), len(shape), d) for d, x in enumerate(xs)], xs


def _kept(v, axes):
    for ax in axes:
        v = v.index_select(ax.d, ax.keep)
    return v


def _grid(axes):
    return tuple(_along(ax.keep, ax.nd, ax.d) for ax in axes)


def _correction(c, axes):
    for ax in reversed(axes):
        c = ax.mass_restrict(c)
    for ax in reversed(axes):
        c = ax.solve(c)
    return c


def _prolonged(z, axes):
    for ax in reversed(axes):
        z = ax.prolong(z)
    return z


def _decomposed(u, coords, levels):
    if levels == 0:
        return u
    axes, xs = _axes(u.shape, coords)
    kept = _kept(u, axes)
    c = u - _prolonged(kept, axes)
    below = _decomposed(kept + _correction(c, axes), [x[ax.keep] for x, ax in zip(xs, axes)], levels - 1)
    return c.index_put(_grid(axes), below)


def _recomposed(y, coords, levels):
    if levels == 0:
        return y
    axes, xs = _axes(y.shape, coords)
    kept = _kept(y, axes)
    c = y.index_put(_grid(axes), torch.zeros_like(kept))
    above = _recomposed(kept, [x[ax.keep] for x, ax in zip(xs, axes)], levels - 1)
    return c + _prolonged(above - _correction(c, axes), axes)


def exact(case, seed):
    kind, dtype = case["kind"], DTYPE[case["dtype"]]
    if kind == "batch":
        return [_decomposed(_field(s, dtype, seed * 1000 + f).double(), None, _full_levels(s))
                for f, s in enumerate(_batch_shapes(case))]
    if kind == "save":  # integers: what a rounding to an integer gives has no value between
        return None
    shape, levels, coords = _shape(case), _levels(case), _coords(case)
    if kind == "load":
        level = max(0, levels - case["drop"])
        codes = _codes(shape, dtype, levels, seed)
        sub, bins = _coarser(shape, levels - level), _bins(shape, levels)
        y, cls = torch.empty(sub, device=DEV, dtype=torch.float64), _classes(sub, level)
        end = 0
        for c in range(level + 1):
            at = cls == c
            n = int(at.sum())
            y[at] = codes[end:end + n].double() * torch.tensor(float(bins[c]), dtype=dtype).item()
            end += n
        return _recomposed(y, None, level)
    if kind == "dec":
        return _decomposed(_field(shape, dtype, seed).double(), coords, levels)
    if kind == "rec":
        return _recomposed(_refactored(shape, dtype, levels, seed).double(), coords, levels)
    if kind == "step":
        x = _field(shape, dtype, seed).double()
        return _decomposed(x, coords, levels), x
    x = (_field(shape, dtype, seed) if kind == "grad" else _refactored(shape, dtype, levels, seed)).double()
    x.requires_grad_(True)
    y = _decomposed(x, coords, levels) if kind == "grad" else _recomposed(x, coords, levels)
    g, = torch.autograd.grad(y, x, _field(shape, dtype, seed + 500009).double())
    return y.detach(), g
