"""Four-way records whose children are opened by box surface: meshes of very
unequal triangles and long chains (where the tree is as deep as its bound
allows and records open down one side), leaves of several triangles and
meshes smaller than a record, against the oracle and the binary walk."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2209_02878_amd import rsi
from tests import parity

pytestmark = pytest.mark.gpu


def _t(a, dtype=torch.float32):
    return torch.as_tensor(np.ascontiguousarray(a)).to(device="cuda", dtype=dtype).contiguous()


def _mesh(kind, n, rng):
    if kind == "chain":  # centroids at 2^-k: one Morton bit per level
        c = 2.0 ** -np.arange(n, dtype=np.float64)[:, None, None] * np.ones((1, 1, 3))
        size = 0.3 * c
    elif kind == "sizes":  # triangles from 1e-4 to the whole box
        c, size = rng.uniform(0, 1, (n, 1, 3)), 10.0 ** rng.uniform(-4, 0, (n, 1, 1))
    else:  # equal centroids: the tree follows the indices
        c, size = np.full((n, 1, 3), 0.5), rng.uniform(0.05, 0.5, (n, 1, 1))
    V = c + size * rng.normal(size=(n, 3, 3))
    if kind == "equal":
        V += 0.5 - V.mean(1, keepdims=True)
    return V.reshape(-1, 3).astype(np.float32), np.arange(3 * n, dtype=np.int32).reshape(n, 3)


@pytest.mark.parametrize("leaf_size", [1, 3])
@pytest.mark.parametrize("kind,n", [("chain", 2), ("chain", 5), ("chain", 60), ("sizes", 7), ("sizes", 3000),
                                    ("equal", 2), ("equal", 600), ("equal", 5000)])
def test_unequal_children(kind, n, leaf_size):
    rng = np.random.default_rng(n)
    V, T = _mesh(kind, n, rng)
    S, E = (rng.uniform(-0.3, 1.3, (2_000, 3)).astype(np.float32) for _ in range(2))
    if kind == "chain":  # towards the small end of the chain
        E[::2] = (rng.uniform(-1, 1, (1_000, 3)) * 2.0 ** -rng.integers(0, 30, (1_000, 1))).astype(np.float32)
    four = rsi.Mesh(_t(V), _t(T, torch.int32), leaf_size=leaf_size, stack_depth=4)
    two = rsi.Mesh(_t(V), _t(T, torch.int32), leaf_size=leaf_size, branching=2)
    ref = parity.oracle_reference(V, T, S, E)
    ok = ref["degenerate"] == 0
    # (the long chain's triangles end below FP32 resolution: both walks then
    # decide alike, but not as the oracle does)
    exact = (kind, n) != ("chain", 60)
    for mode in ("bool", "first", "count"):
        a, b = four.query(_t(S), _t(E), mode), two.query(_t(S), _t(E), mode)
        st = four.stats()
        assert st["stack_dropped"] == 0 and st["walk_cut"] == 0
        if mode == "count" and exact:
            assert np.array_equal(a["count"].cpu().numpy()[ok], ref["count"][ok])
        elif mode == "first" and exact:
            assert np.array_equal(a["tri"].cpu().numpy()[ok], ref["first_tri"][ok])
        for k in a:
            x, y = a[k].cpu().numpy()[ok], b[k].cpu().numpy()[ok]
            assert np.array_equal(x, y), (mode, k)
    four.close()
    two.close()
