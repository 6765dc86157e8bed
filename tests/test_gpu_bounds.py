"""Bounding boxes reduced in registers: centroid bounds of meshes around the
eight-triangles-per-thread limit and of batches whose mesh borders fall
inside a thread's, a wave's and a workgroup's triangles, and midpoint bounds
of segment arrays with every alignment and remainder.  The Morton codes and
orders that follow from the boxes are held to numpy."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2209_02878_amd import rsi
from tests.test_gpu_order import host_keys

pytestmark = pytest.mark.gpu


def _t(a, dtype=torch.float32):
    return torch.as_tensor(np.ascontiguousarray(a)).to(device="cuda", dtype=dtype).contiguous()


def _soup(n, rng):
    c = rng.normal(size=(n, 1, 3)) * rng.uniform(0.5, 20) + rng.uniform(-50, 50, 3)
    V = (c + 0.1 * rng.normal(size=(n, 3, 3))).reshape(-1, 3).astype(np.float32)
    return V, np.arange(3 * n, dtype=np.int32).reshape(n, 3)


def _codes(V, T):
    P = V[T]
    c = ((P[:, 0] + P[:, 1]).astype(np.float32) + P[:, 2]).astype(np.float32) * np.float32(1.0 / 3.0)
    lo, hi = c.min(0), c.max(0)
    ext = (hi - lo).astype(np.float32)
    code = np.zeros(len(c), np.uint64)
    for k in range(3):
        q = np.zeros(len(c), np.uint64)
        if ext[k] > 0:
            x = ((c[:, k] - lo[k]).astype(np.float32) / ext[k]).astype(np.float32) * np.float32(2097152.0)
            q = np.clip(x, 0, 2097151).astype(np.uint64)
        for b in range(21):
            code |= ((q >> np.uint64(b)) & np.uint64(1)) << np.uint64(3 * b + 2 - k)
    return code


@pytest.mark.parametrize("n", [1, 255, 257, 131_071, 131_072, 131_073, 140_001])
def test_centroid_bounds(n):
    V, T = _soup(n, np.random.default_rng(n))
    mesh = rsi.Mesh(_t(V), _t(T, torch.int32))
    assert np.array_equal(mesh.tree()["keys"], np.sort(_codes(V, T)))
    mesh.close()


def test_centroid_bounds_of_batches():
    rng = np.random.default_rng(5)
    sizes = [1, 3, 100, 255, 256, 257, 2047, 2, 2, 2, 2, 2, 2, 2049, 70_000, 64, 65, 60_000]
    meshes = [_soup(n, rng) for n in sizes]
    batch = rsi.Batch([(_t(V), _t(T, torch.int32)) for V, T in meshes])
    keys, at = batch.tree()["keys"], 0
    for (V, T), n in zip(meshes, sizes):
        assert np.array_equal(keys[at:at + n], np.sort(_codes(V, T))), n
        at += n
    batch.close()


@pytest.mark.parametrize("shift", [0, 1, 2, 3])
@pytest.mark.parametrize("n", [1, 2, 3, 5, 1279, 1280, 1281, 400_003])
def test_segment_bounds_alignment(n, shift):
    """Arrays that start `shift` rows (12 bytes each) into an allocation."""
    rng = np.random.default_rng(n + shift)
    S, E = (rng.normal(size=(n, 3)).astype(np.float32) * np.float32(3) + np.float32(k) for k in (-7, 11))
    V, T = _soup(4, rng)
    mesh = rsi.Mesh(_t(V), _t(T, torch.int32))
    St, Et = (torch.cat([torch.full((shift, 3), 1e9, device="cuda"), _t(x)])[shift:] for x in (S, E))
    order, So, Eo = mesh.segment_order(St, Et)
    assert np.array_equal(order.cpu().numpy(), np.argsort(host_keys(S, E), kind="stable"))
    assert torch.equal(So, St[order.long()]) and torch.equal(Eo, Et[order.long()])
    mesh.close()


@pytest.mark.parametrize("each", [7, 63, 64, 65, 190])
def test_centroid_bounds_of_many_small_meshes(each):
    """A workgroup of the eight-per-thread pass spans 2,048 triangles and keeps
    32 meshes in LDS: borders below, at and above that, meshes of one triangle
    and larger ones among them."""
    rng = np.random.default_rng(each)
    sizes = [each + (k % 3) for k in range(135_000 // each)]
    sizes[10:10] = [1] * 40
    sizes[90:90] = [5_000]
    parts = [_soup(n, rng) for n in sizes]
    batch = rsi.Batch([(_t(V), _t(T, torch.int32)) for V, T in parts])
    keys, at = batch.tree()["keys"], 0
    for (V, T), n in zip(parts, sizes):
        assert np.array_equal(keys[at:at + n], np.sort(_codes(V, T))), n
        at += n
    batch.close()
