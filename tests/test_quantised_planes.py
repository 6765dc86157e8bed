"""The planes of the four-way records, placed in FP64 as Wide::store does: each
is on the grid and outside its child's box by at least the 2^-11 steps that
the box test relies on (or the node's corner), for every finite box, extents
past the FP32 range among them, and not a whole step further out; and the
box test of test_qslab_conservative.py rejects no touched box with them."""
from fractions import Fraction

import numpy as np
import pytest

import tests.test_qslab_conservative as q

MARGIN = 2.0 ** -11 + 2.0 ** -40


def grid64(lo, hi):
    """Steps of a node whose box is [lo, hi]: the exponent of the next power
    of two above extent / (255 - 2^-10), from the bits of the FP64 value."""
    step = []
    for k in range(3):
        x = (np.float64(hi[k]) - np.float64(lo[k])) * ((1 + 2.0 ** -40) / (255 - 2.0 ** -10))
        u = int(np.float64(x).view(np.uint64))
        e = (u >> 52) - 1023 + (1 if u & ((1 << 52) - 1) else 0) if x > 2.0 ** -126 else -126
        step.append(2.0 ** min(e, 127))
    return step


def planes64(lo, step, clo, chi):
    qlo, qhi = [], []
    for k in range(3):
        inv = 1.0 / step[k]
        at = (np.float64(clo[k]) - np.float64(lo[k])) * inv, (np.float64(chi[k]) - np.float64(lo[k])) * inv
        # to nearest (even), after a move by half a step and the margin
        qlo.append(int(min(max(np.rint(at[0] - 0.5 - MARGIN), 0), 255)))
        qhi.append(int(min(max(np.rint(at[1] + 0.5 + MARGIN), 0), 255)))
        corner, st = Fraction(float(lo[k])), Fraction(step[k])
        lower, upper = corner + qlo[k] * st, corner + qhi[k] * st
        assert qlo[k] == 0 or lower <= Fraction(float(clo[k])) - st / 2048
        assert lower <= Fraction(float(clo[k])) and upper >= Fraction(float(chi[k])) + st / 2048
        # and no looser than the grid and the margin make it
        assert lower > Fraction(float(clo[k])) - st * Fraction(2050, 2048)
        assert upper < Fraction(float(chi[k])) + st * Fraction(2050, 2048)
    return qlo, qhi


@pytest.mark.parametrize("size", [0.0, 1e-45, 1e-40, 1e-30, 1e-3, 1.0, 1e20, 3.4e38])
def test_planes_of_any_finite_box(size):
    rng = np.random.default_rng(3)
    for _ in range(400):
        far = 0.0 if size > 1e30 or rng.uniform() < 0.5 else size * 10.0 ** rng.uniform(0, 7)
        a, b = ((far + rng.uniform(-size, size, (2, 3))).astype(np.float32) for _ in range(2))
        lo, hi = np.minimum(a.min(0), b.min(0)), np.maximum(a.max(0), b.max(0))
        planes64(lo, grid64(lo, hi), a.min(0), a.max(0))


def test_extent_past_the_fp32_range():
    """The second child starts near the middle of a box 6.8e38 wide: its lower
    plane lies there, not at the far side."""
    lo, hi = np.full(3, -3.4e38, np.float32), np.full(3, 3.4e38, np.float32)
    step = grid64(lo, hi)
    assert 255 * step[0] >= 6.8e38 > 126 * step[0]
    qlo, qhi = planes64(lo, step, np.zeros(3, np.float32), hi)
    assert qlo[0] == 63 and qhi[0] == 128


@pytest.mark.parametrize("case", [q.test_random_segments, q.test_flat_boxes_and_axis_parallel_segments,
                                  q.test_cut_segments_keep_what_the_cut_reaches,
                                  lambda: q.test_ends_on_faces(1.0), lambda: q.test_ends_on_faces(1e4),
                                  lambda: q.test_other_scales(1e-30), lambda: q.test_other_scales(1e-6),
                                  lambda: q.test_other_scales(1e6), lambda: q.test_other_scales(1e12)])
def test_box_test_with_these_planes(case, monkeypatch):
    monkeypatch.setattr(q, "grid", grid64)
    monkeypatch.setattr(q, "planes", planes64)
    case()
