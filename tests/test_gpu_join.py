"""Subtrees that cross the local build blocks, joined in LDS.

The local pass completes subtrees inside blocks of 512 sorted leaves (2,048
where one block holds the mesh); one workgroup joins what up to 64 blocks
leave, and a further one what those leave.  Sizes here lie on either side of a
block, of 64 blocks, of 256 and of the change of block size; the chain's centroids halve from one
triangle to the next (the deepest paths a key allows), with enough copies of
each that the path crosses blocks.  The trees are held to the exact validator
of test_gpu_tree.py, after a build and after a refit.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2209_02878_amd import rsi
from tests.test_gpu_tree import _mesh, _validate

pytestmark = pytest.mark.gpu


def _soup(centers, size):
    rng = np.random.default_rng(len(centers))
    V = (centers[:, None, :] + rng.uniform(-size, size, (len(centers), 3, 3))).astype(np.float32).reshape(-1, 3)
    return V, np.arange(len(V), dtype=np.int32).reshape(-1, 3)


@pytest.mark.parametrize("n,leaf", [(513, 1), (2049, 4), (32_768, 1), (32_769, 16), (131_072, 1), (131_073, 1)])
def test_blocks(n, leaf):
    rng = np.random.default_rng(n)
    V, T = _soup(rng.uniform(0, 1, (n, 3)) ** 2, 1e-3)
    m = _mesh(V, T, leaf_size=leaf)
    inner = _validate(m.tree(), V, T, leaf)
    assert leaf > 1 or inner == n - 1
    W = (V * np.float32(1.5)).astype(np.float32)
    m.refit(torch.from_numpy(W).cuda())
    _validate(m.tree(), W, T, leaf)
    m.close()


@pytest.mark.parametrize("copies", [11, 97, 2100])
def test_chain(copies):
    k = np.repeat(np.arange(22), copies)
    V, T = _soup(np.stack([0.5 ** k, 0.5 ** k, 0.5 ** k], 1), 1e-9)
    m = _mesh(V, T)
    _validate(m.tree(), V, T, 1)
    m.close()


def test_meshes_across_blocks():
    """A batch whose meshes begin and end inside blocks: each one's tree is
    that of a handle of its own, so the first hits are the same."""
    rng = np.random.default_rng(8)
    sizes = [1, 700, 3, 2048, 5000, 40_000, 511, 30_001, 2]
    meshes, singles, ends = [], [], []
    for n in sizes:
        V, T = _soup(rng.uniform(0, 1, (n, 3)), 0.02)
        meshes.append((torch.from_numpy(V).cuda(), torch.from_numpy(T).cuda()))
        singles.append(rsi.Mesh(*meshes[-1]))
        ends.append(tuple(torch.from_numpy(rng.uniform(0, 1, (500, 3)).astype(np.float32)).cuda() for _ in range(2)))
    b = rsi.Batch(meshes)
    out = b.query(ends, "first")
    for x, m, (S, E) in zip(out, singles, ends):
        y = m.query(S, E, "first")
        for key in ("tri", "t", "uv", "point"):
            assert torch.equal(x[key], y[key]), key
        m.close()
    b.close()


@pytest.mark.parametrize("n,leaf", [(511, 1), (512, 3), (1399, 1), (1400, 1), (1401, 1), (1536, 2), (1537, 1),
                                    (2047, 1), (2048, 16)])
def test_one_block_or_blocks_of_512(n, leaf):
    """Up to 1,400 triangles one block holds the mesh."""
    rng = np.random.default_rng(n)
    V, T = _soup(rng.uniform(0, 1, (n, 3)) ** 2, 1e-3)
    m = _mesh(V, T, leaf_size=leaf)
    inner = _validate(m.tree(), V, T, leaf)
    assert leaf > 1 or inner == n - 1
    W = (V * np.float32(1.5)).astype(np.float32)
    m.refit(torch.from_numpy(W).cuda())
    _validate(m.tree(), W, T, leaf)
    m.close()
