"""The sort's last pass at the sizes where it can go wrong: groups of equal
key prefixes around the window's halo (512 keys) and far past it,
keys equal throughout (the order must stay stable), and totals around the
changes of the number of digit passes.  Held bit for bit to a stable host
sort of the same keys, through the segment order; the Morton order of a
clustered batch is held to single builds."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2209_02878_amd import rsi
from paper_2209_02878_amd import workloads as wl
from tests.test_gpu_order import host_keys
from tests.test_gpu_tree import _morton_reference

pytestmark = pytest.mark.gpu


def _t(a, dtype=torch.float32):
    return torch.as_tensor(np.ascontiguousarray(a)).to(device="cuda", dtype=dtype).contiguous()


def _order(S, E):
    V, T = wl.noisy_sphere(2, 5, 0.3)
    mesh = rsi.Mesh(_t(V), _t(T, torch.int32))
    order, _, _ = mesh.segment_order(_t(S), _t(E))
    got = order.cpu().numpy()
    mesh.close()
    return got


def _clusters(sizes, width, rng):
    """Segments whose midpoints crowd into one small cube per entry of
    `sizes` (shuffled), a few far ones setting the box."""
    mids = [np.array([[0, 0, 0], [1, 1, 1]], np.float64)]
    for s in sizes:
        mids.append(rng.uniform(0.05, 0.95, 3) + width * rng.uniform(-1, 1, (s, 3)))
    m = np.concatenate(mids)
    m = m[rng.permutation(len(m))]
    d = rng.uniform(0.001, 0.002, 3)
    return (m - d).astype(np.float32), (m + d).astype(np.float32)


@pytest.mark.parametrize("width", [0.0, 1e-3, 8e-3])
@pytest.mark.parametrize("sizes", [
    [511, 512, 513, 1023, 1025, 2500, 1, 7],                         # one pass
    [511, 512, 513, 1025, 2047, 2049, 4097, 30_000, 1] + [600] * 20,  # two passes, tiles of 256
    [511, 512, 513, 1025, 2047, 2049, 70_000, 3] + [515] * 200,       # two passes, tiles of 2,048
])
def test_clustered_segments(sizes, width):
    rng = np.random.default_rng(len(sizes))
    S, E = _clusters(sizes, width, rng)
    assert np.array_equal(_order(S, E), np.argsort(host_keys(S, E), kind="stable"))


@pytest.mark.parametrize("n", [2, 255, 256, 257, 1023, 1024, 1025, 16_384, 16_385, 32_768, 32_769, 131_072, 131_073, 1_048_577])
def test_totals_around_the_plan_changes(n):
    rng = np.random.default_rng(n)
    S, E = wl.segments_in_box(rng, [0, 0, 0], [1, 1, 0.1], n)
    assert np.array_equal(_order(S, E), np.argsort(host_keys(S, E), kind="stable"))


def test_clustered_batch_matches_single_builds():
    rng = np.random.default_rng(3)
    meshes = []
    for n_t, spread in ((1, 1.0), (900, 0.0), (3_000, 1e-4), (1_300, 1e-7), (70_000, 1e-3), (2, 1.0)):
        c = rng.uniform(0, 1, (n_t, 1, 3)) * spread + rng.integers(0, 2, (n_t, 1, 3))
        V = (c + 0.01 * rng.uniform(-1, 1, (n_t, 3, 3)) * (spread > 0)).reshape(-1, 3).astype(np.float32)
        meshes.append((_t(V), _t(np.arange(3 * n_t).reshape(n_t, 3), torch.int32)))
    batch = rsi.Batch(meshes)
    tree, base = batch.tree(), 0
    for V, T in meshes:
        m = rsi.Mesh(V, T)
        one, n = m.tree(), T.shape[0]
        assert np.array_equal(tree["order"][base:base + n] - base, one["order"])
        assert np.array_equal(tree["keys"][base:base + n], one["keys"])
        assert np.array_equal(np.argsort(one["keys"], kind="stable"), np.arange(n))
        same = one["keys"][1:] == one["keys"][:-1]
        assert np.all(one["order"][1:][same] > one["order"][:-1][same])
        base += n
        m.close()
    batch.close()


@pytest.mark.parametrize("meshes,each", [(2, 8000), (9, 1800), (70, 400), (3, 10_900)])
def test_few_and_many_mesh_ids(meshes, each):
    """Tables of at most 16 tiles count the mesh id's digits in the pass before:
    lanes that agree add together, down to groups of eight."""
    rng = np.random.default_rng(meshes)
    parts = []
    for m in range(meshes):
        c = rng.uniform(0, 1, (each + 7 * m, 1, 3)) + rng.uniform(-0.01, 0.01, (each + 7 * m, 3, 3))
        V = c.astype(np.float32).reshape(-1, 3)
        parts.append((V, np.arange(len(V), dtype=np.int32).reshape(-1, 3)))
    b = rsi.Batch([(torch.from_numpy(V).cuda(), torch.from_numpy(T).cuda()) for V, T in parts])
    tree = b.tree()
    at = 0
    for V, T in parts:
        ref = _morton_reference(V, T)
        want = np.argsort(ref, kind="stable")
        n = len(T)
        assert np.array_equal(tree["keys"][at:at + n], ref[want])
        assert np.array_equal(tree["order"][at:at + n] - at, want)
        at += n
    b.close()


@pytest.mark.parametrize("size", [513, 1024, 1025, 2048, 2049, 4096, 4097])
@pytest.mark.parametrize("spread", [0.0, 1e-6, 1e-3])
def test_far_triangle(size, spread):
    """One far triangle puts all others in one group of equal top bits: sizes
    around those sorted in LDS by 4, 8 and 16 keys a thread, or past it, with
    63-bit keys; beside small groups in tables of other tiles."""
    rng = np.random.default_rng(size)
    for rest in (0, 150_000):  # far more triangles: the large tiles
        c = np.concatenate([0.3 + spread * rng.uniform(-1, 1, (size, 1, 3)), [[[9.0, 9.0, 9.0]]],
                            rng.uniform(4, 8, (rest, 1, 3))])
        V = (c + 1e-3 * spread * rng.uniform(-1, 1, (len(c), 3, 3))).astype(np.float32).reshape(-1, 3)
        T = rng.permutation(len(c)).astype(np.int32)[:, None] * 3 + np.arange(3, dtype=np.int32)
        mesh = rsi.Mesh(_t(V), _t(T, torch.int32))
        tree = mesh.tree()
        ref = _morton_reference(V, T)
        want = np.argsort(ref, kind="stable")
        assert np.array_equal(tree["keys"], ref[want])
        assert np.array_equal(tree["order"], want)
        mesh.close()


@pytest.mark.parametrize("n", [4_194_304, 4_194_305, 5_000_011])
@pytest.mark.parametrize("width", [0.0, 1e-6, 1e-3])
def test_far_segment_in_a_large_table(n, width):
    """Above 2^22 keys a group of more than 16,384 equal prefixes is sorted by
    passes over the whole table."""
    rng = np.random.default_rng(n)
    S, E = _clusters([n - 20_000, 10_000, 9_998], width, rng)
    assert len(S) == n
    assert np.array_equal(_order(S, E), np.argsort(host_keys(S, E), kind="stable"))


@pytest.mark.parametrize("meshes", [1, 2, 300])
def test_far_triangle_in_a_large_table(meshes):
    """The same with 63-bit keys, alone and under one or two mesh-id digits."""
    rng = np.random.default_rng(meshes)
    sizes = [4_300_000] + [50 + k for k in range(meshes - 1)]
    parts = []
    for n in sizes:
        c = (0.3 + 1e-4 * rng.uniform(-1, 1, (n, 1, 3))).astype(np.float32)
        c[0] = 9
        V = (c + 1e-5 * rng.uniform(-1, 1, (n, 3, 3))).astype(np.float32).reshape(-1, 3)
        parts.append((_t(V), _t(np.arange(3 * n).reshape(n, 3), torch.int32)))
    mesh = rsi.Batch(parts) if meshes > 1 else rsi.Mesh(*parts[0])
    tree, at = mesh.tree(), 0
    for (V, T), n in zip(parts, sizes):
        ref = _morton_reference(V.cpu().numpy(), T.cpu().numpy())
        want = np.argsort(ref, kind="stable")
        assert np.array_equal(tree["keys"][at:at + n], ref[want])
        assert np.array_equal(tree["order"][at:at + n] - at, want)
        at += n
    mesh.close()


def test_time_of_a_large_table_with_one_far_segment():
    """Not left to a few workgroups: 4.8 times the time without the far segment
    when it was, about twice with the passes over the whole table."""
    n = 5_000_000
    S = torch.rand(n, 3, device="cuda", generator=torch.Generator("cuda").manual_seed(1))
    E = S + 0.01
    far = S * 1e-3
    far[0] = 5
    V, T = wl.noisy_sphere(2, 5, 0.3)
    mesh = rsi.Mesh(_t(V), _t(T, torch.int32))
    times = []
    for s, e in ((S, E), (far, far + 1e-5)):
        ms = []
        for _ in range(4):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            mesh.segment_order(s, e)
            b.record()
            torch.cuda.synchronize()
            ms.append(a.elapsed_time(b))
        times.append(min(ms))
    mesh.close()
    assert times[1] < 3.5 * times[0], times


@pytest.mark.parametrize("n", [20_480, 20_481])
@pytest.mark.parametrize("flat", [False, True])
def test_totals_around_the_short_keys_limit(n, flat):
    """Segments' 33-bit keys: one pass up to 20,480, then two; spread over a
    volume, and with every midpoint on a plane (groups of over 512 keys)."""
    rng = np.random.default_rng(n)
    S, E = wl.segments_in_box(rng, [0, 0, 0], [1, 1, 0.1], n)
    if flat:
        S[:, 2], E[:, 2] = 1.0, -1.0
    assert np.array_equal(_order(S, E), np.argsort(host_keys(S, E), kind="stable"))


def test_totals_around_the_triangles_limits():
    """63-bit codes: one pass up to 16,384 triangles, two up to 262,144."""
    rng = np.random.default_rng(7)
    for n in (16_384, 16_385, 262_144, 262_145):
        c = rng.uniform(0, 1, (n, 1, 3)) * np.array([1, 1, 0.05])
        V = (c + 1e-4 * rng.uniform(-1, 1, (n, 3, 3))).astype(np.float32).reshape(-1, 3)
        T = np.arange(3 * n, dtype=np.int32).reshape(n, 3)
        mesh = rsi.Mesh(_t(V), _t(T, torch.int32))
        ref = _morton_reference(V, T)
        want = np.argsort(ref, kind="stable")
        tree = mesh.tree()
        assert np.array_equal(tree["keys"], ref[want]) and np.array_equal(tree["order"], want), n
        mesh.close()
