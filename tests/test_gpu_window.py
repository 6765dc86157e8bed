"""The four-way walk's stack window: entries past the LDS part move to device
memory in halves and come back.  Window sizes from one entry to past the
deepest stack, in every mode, must give the default's answers bit for bit
(which the parity tests hold to the oracle)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2209_02878_amd import rsi
from paper_2209_02878_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _t(a, dtype=torch.float32):
    return torch.as_tensor(np.ascontiguousarray(a)).to(device="cuda", dtype=dtype).contiguous()


@pytest.mark.parametrize("n", [20_011, 700_001])  # fewer segments than lanes (walks shared), and more
@pytest.mark.parametrize("depth", [1, 3, 5, 6, 9, 255])
def test_window_sizes_keep_answers(depth, n):
    V, T = wl.noisy_sphere(30, 4, 0.3)
    S, E = wl.segments_in_box(np.random.default_rng(9), V.min(0), V.max(0), n, scale=1.5)
    V, T, S, E = _t(V), _t(T, torch.int32), _t(S), _t(E)
    base, small = rsi.Mesh(V, T), rsi.Mesh(V, T, stack_depth=depth)
    for mode in ("bool", "first", "count", "all", "first|count", "all|first|bool"):
        want, got = base.query(S, E, mode, capacity=2), small.query(S, E, mode, capacity=2)
        st = small.stats()
        assert st["stack_dropped"] == 0 and st["walk_cut"] == 0
        if depth <= 3:
            assert st["deep_segments"] > 0, mode
        for k in want:
            if k != "spill":
                assert torch.equal(want[k], got[k]), (mode, k)
    base.close()
    small.close()


@pytest.mark.parametrize("n", [1, 232, 233])
@pytest.mark.parametrize("depth", [1, 9])
def test_launch_with_a_column_for_each_lane(depth, n):
    """Up to 232 segments every lane has a stack column in device memory and no
    deep pass follows; the answers are those of the same segments in a larger
    launch with the default window."""
    V, T = wl.noisy_sphere(30, 4, 0.3)
    S, E = wl.segments_in_box(np.random.default_rng(10), V.min(0), V.max(0), n, scale=1.5)
    V, T, S, E = _t(V), _t(T, torch.int32), _t(S), _t(E)
    many = rsi.Mesh(V, T)
    small = rsi.Mesh(V, T, stack_depth=depth)
    reps = 4000 // n + 1
    for mode in ("bool", "first", "count", "all"):
        # the same segments among so many that the deep pass is launched
        want = many.query(S.repeat(reps, 1), E.repeat(reps, 1), mode, capacity=2)
        got = small.query(S, E, mode, capacity=2)
        st = small.stats()
        assert st["stack_dropped"] == 0 and st["walk_cut"] == 0
        for k in got:
            if k not in ("spill", "spill_off"):
                assert torch.equal(want[k][: got[k].shape[0]], got[k]), (mode, k)
    many.close()
    small.close()


@pytest.mark.parametrize("n", [1, 3, 70, 2_000])
def test_overflowed_segments_are_counted_once(n):
    """deep_segments counts segments, however many lanes walked parts of one and
    whichever of them overflowed: upright segments through 2,000 sheets."""
    k = np.arange(2_000, dtype=np.float32)[:, None, None] / 2_000
    quad = np.array([[0, 0, 0], [1, 0, 0], [1, 1, 0], [0, 1, 0]], np.float32)
    V = (quad + k * np.array([0, 0, 1], np.float32)).reshape(-1, 3)
    T = (4 * np.arange(2_000)[:, None, None] + np.array([[0, 1, 2], [0, 2, 3]])).reshape(-1, 3)
    xy = np.random.default_rng(12).uniform(0.1, 0.9, (n, 2)).astype(np.float32)
    S, E = (_t(np.concatenate([xy, np.full((n, 1), z, np.float32)], 1)) for z in (-1.0, 2.0))
    small = rsi.Mesh(_t(V), _t(T, torch.int32), stack_depth=3)
    for mode in ("count", "all", "first|count"):
        got = small.query(S, E, mode, capacity=2)
        assert torch.all(got["count"] >= 2_000)
        st = small.stats()
        assert st["deep_segments"] == n, (mode, st)
    small.close()
