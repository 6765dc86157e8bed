"""The quantised box test of the four-way walk never rejects a box that the
segment touches.

Restates, in FP32 through numpy, the grid of a node (Wide::store: corner,
power-of-two steps, child planes at least 2^-11 steps outside the child's
box except a lower plane at the corner), the guarded reciprocal (box_tiny,
box_rcp; the hardware reciprocal taken as any value within 1 ulp) and the
test itself (qslab_hit: planes at fma(q, a, b -+ |b| 2^-19), shifted by
2^-21, clamped to [0, 1], near < far), and holds it to the exact rational
slab test of test_slab_conservative.py.  fma is formed in FP64 and rounded
once; the product of two FP32 numbers is exact there.
"""
from fractions import Fraction

import numpy as np
import pytest

from tests.test_slab_conservative import F32, _box, exact_touch

_rng = np.random.default_rng(3)


def fma(a, b, c):
    return F32(np.float64(a) * np.float64(b) + np.float64(c))


def grid(lo, hi):
    """Steps of a node whose box is [lo, hi]: the exponent of the next power
    of two above extent / 254.5, from the bits of the FP32 value."""
    step = []
    for k in range(3):
        x = F32(F32(hi[k] - lo[k]) * F32((1 + 2.0 ** -20) / 254.5))
        u = int(x.view(np.uint32))
        e = (u >> 23) - 127 + (1 if u & 0x7FFFFF else 0)
        step.append(2.0 ** min(max(e, -126), 127))
    return step


def planes(lo, step, clo, chi):
    qlo, qhi = [], []
    for k in range(3):
        inv, m = F32(1.0 / step[k]), F32(2.0 ** -10)
        x = np.floor(F32(F32(F32(clo[k] - lo[k]) * inv) - m))
        y = np.ceil(F32(F32(F32(chi[k] - lo[k]) * inv) + m))
        qlo.append(int(min(max(x, 0), 255)))
        qhi.append(int(min(max(y, 0), 255)))
        # the quantised box holds the child's (exactly), and by the margin the
        # box test needs wherever a plane is not the corner itself
        assert Fraction(qhi[k]) * Fraction(step[k]) + Fraction(float(lo[k])) >= Fraction(float(chi[k])) + Fraction(
            step[k]) / 2048
        assert qlo[k] == 0 or Fraction(qlo[k]) * Fraction(step[k]) + Fraction(float(lo[k])) <= Fraction(
            float(clo[k])) - Fraction(step[k]) / 2048
    return qlo, qhi


def accepts(s, e, lo, hi, clo, chi, tlim=F32(1.0)):
    """The test of child box [clo, chi] in a node whose box is [lo, hi], the
    mesh's box being the node's."""
    step = grid(lo, hi)
    qlo, qhi = planes(lo, step, clo, chi)
    d = (e - s).astype(F32)
    scale = F32(np.max(np.abs(np.concatenate([lo, hi]))))
    R = F32(scale + F32(np.max(np.abs(s))))
    tiny = fma(R, F32(2.0 ** -125), F32(2.0 ** -126))
    near, far = F32(-np.inf), F32(np.inf)
    for k in range(3):
        g = np.copysign(np.maximum(F32(np.abs(d[k]) * tlim), tiny), d[k]).astype(F32)
        inv = F32(F32(1.0) / g)
        move = _rng.integers(-1, 2)
        if move:
            inv = np.nextafter(inv, F32(np.inf) if move > 0 else F32(-np.inf)).astype(F32)
        a = F32(F32(step[k]) * inv)
        b = fma(F32(F32(lo[k]) - s[k]), inv, F32(2.0 ** -21))
        bn, bf = fma(-abs(b), F32(2.0 ** -19), b), fma(abs(b), F32(2.0 ** -19), b)
        assert np.isfinite([a, b, bn, bf]).all()
        qn, qf = (qlo[k], qhi[k]) if inv >= 0 else (qhi[k], qlo[k])
        near, far = max(near, fma(F32(qn), a, bn)), min(far, fma(F32(qf), a, bf))
    return min(max(near, F32(0)), F32(1)) < min(max(far, F32(0)), F32(1))


def _check(cases):
    touched = kept = 0
    for s, e, lo, hi, clo, chi in cases:
        ok, face = exact_touch(s, e, clo, chi)
        acc = accepts(s, e, lo, hi, clo, chi)
        if ok and not face and np.any(e != s):
            touched += 1
            assert acc, (s, e, lo, hi, clo, chi)
        kept += acc
    return touched, kept


def _node(rng, c, size):
    """A node's box, and a child's box inside it that shares some faces."""
    lo, hi = _box(rng, c, size)
    u, v = _box(rng, c, size)
    clo, chi = np.clip(u, lo, hi), np.clip(v, lo, hi)
    for k in range(3):
        if rng.uniform() < 0.3:
            clo[k] = lo[k]
        if rng.uniform() < 0.3:
            chi[k] = hi[k]
    return lo, hi, clo, chi


def test_random_segments():
    rng = np.random.default_rng(1)
    cases = []
    for _ in range(3000):
        c = rng.uniform(-1, 1, 3) * (1000.0 if rng.uniform() < 0.2 else 1.0)
        box = _node(rng, c, 10.0 ** rng.uniform(-4, -0.3))
        s = (c + rng.uniform(-0.6, 0.6, 3)).astype(F32)
        e = (rng.uniform(box[2], box[3]) + rng.normal(size=3) * rng.uniform(0, 0.3)).astype(F32)
        cases.append((s, e, *box))
    touched, kept = _check(cases)
    assert touched > 50 and kept < 3000  # and it still rejects


@pytest.mark.parametrize("far", [1.0, 1e4])
def test_ends_on_faces(far):
    """A start or an end exactly on a face of the child's box, the node's
    corner among them: near or far is then exactly the end of the range."""
    rng = np.random.default_rng(2)
    cases = []
    for _ in range(3000):
        box = _node(rng, rng.uniform(-1, 1, 3) * far, 10.0 ** rng.uniform(-3, -0.5))
        p = rng.uniform(box[2], box[3]).astype(F32)
        p = np.clip(p, box[2], box[3])
        for k in range(3):
            if rng.uniform() < 0.5:
                p[k] = box[2][k] if rng.uniform() < 0.5 else box[3][k]
        q = (p + rng.normal(size=3) * 10.0 ** rng.uniform(-4, 1)).astype(F32)
        cases.append((p, q, *box) if rng.uniform() < 0.5 else (q, p, *box))
    assert _check(cases)[0] > 2000


def test_flat_boxes_and_axis_parallel_segments():
    """Flat nodes and children (a plane of triangles), segments that start on
    the plane, zero and tiny direction components."""
    rng = np.random.default_rng(4)
    cases = []
    for _ in range(3000):
        lo, hi, clo, chi = _node(rng, rng.uniform(-1, 1, 3), 10.0 ** rng.uniform(-3, -0.5))
        k = rng.integers(3)
        hi[k] = lo[k]
        clo[k] = chi[k] = lo[k]
        p = np.clip(rng.uniform(clo, chi).astype(F32), clo, chi)
        d = rng.normal(size=3) * 10.0 ** rng.uniform(-3, 1)
        j = rng.integers(3)
        d[j] *= 0.0 if rng.uniform() < 0.5 else 10.0 ** rng.uniform(-30, -3)
        q = (p + d).astype(F32)
        r = rng.uniform()
        if r < 0.4:
            cases.append((p, q, lo, hi, clo, chi))
        elif r < 0.8:
            cases.append((q, p, lo, hi, clo, chi))
        else:
            cases.append(((p - d).astype(F32), q, lo, hi, clo, chi))
    assert _check(cases)[0] > 800


@pytest.mark.parametrize("scale", [1e-30, 1e-6, 1e6, 1e12])
def test_other_scales(scale):
    rng = np.random.default_rng(6)
    cases = []
    for _ in range(1500):
        box = tuple((x * F32(scale)).astype(F32) for x in _node(rng, rng.uniform(-1, 1, 3), 0.3))
        s = (rng.uniform(-1.5, 1.5, 3) * scale).astype(F32)
        e = (rng.uniform(box[2], box[3]) + rng.normal(size=3) * 0.2 * scale * rng.uniform()).astype(F32)
        if rng.uniform() < 0.3:
            k = rng.integers(3)
            e[k] = s[k]
        cases.append((s, e, *box))
    assert _check(cases)[0] > 150


def test_cut_segments_keep_what_the_cut_reaches():
    """The first-hit walk cuts the segment at tlim: a box met before the cut
    stays."""
    rng = np.random.default_rng(8)
    touched = 0
    for _ in range(2000):
        lo, hi, clo, chi = _node(rng, rng.uniform(-1, 1, 3), 10.0 ** rng.uniform(-3, -0.5))
        p = np.clip(rng.uniform(clo, chi).astype(F32), clo, chi)
        d = rng.normal(size=3)
        tl = 10.0 ** rng.uniform(-3, 0)
        s, e = (p - tl * d).astype(F32), (p + (1 - tl) * d).astype(F32)
        cut = F32(tl * (1 + 2.0 ** -18))
        if exact_touch(s, e, clo, chi, float(cut) * (1 - 2.0 ** -20))[0]:
            touched += 1
            assert accepts(s, e, lo, hi, clo, chi, cut)
    assert touched > 800
