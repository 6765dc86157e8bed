"""The adjoint on small meshes, whose few cells are walked by more workgroups
the more segments there are: one call over all segments against the sum of
calls over parts short enough for the four workgroups that every cell has.

dS and dE are per segment: the same bits.  dV: every part's sum is FP64
rounded once to FP32, so the total is within 2^-24 of the summed magnitudes
for the parts and as much for the one call; twice that is allowed."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2209_02878_amd import rsi
from paper_2209_02878_amd import workloads as wl

pytestmark = pytest.mark.gpu

PART = 4096


def _t(a, dtype=torch.float32):
    return torch.as_tensor(np.ascontiguousarray(a)).to(device="cuda", dtype=dtype).contiguous()


@pytest.mark.parametrize("grid,n", [(3, 10_239), (3, 10_240), (3, 300_001), (24, 61_440), (40, 200_003)])
def test_chunks(grid, n):
    V, T = wl.sinusoid_heightfield(grid, 3, 0.1)
    S, E = wl.segments_near_vertical(np.random.default_rng(n), n)
    g = np.random.default_rng(n + 1)
    gt, guv, gp = g.normal(size=n), g.normal(size=(n, 2)), g.normal(size=(n, 3))
    V, T, S, E, gt, guv, gp = _t(V), _t(T, torch.int32), _t(S), _t(E), _t(gt), _t(guv), _t(gp)
    m = rsi.Mesh(V, T)
    tri = m.query(S, E, "first")["tri"]
    dV, dS, dE = m.first_hit_backward(V, S, E, tri, gt, guv, gp)
    assert torch.equal(dV, m.first_hit_backward(V, S, E, tri, gt, guv, gp)[0])
    total = torch.zeros_like(dV, dtype=torch.float64)
    size = torch.zeros_like(total)
    for i in range(0, n, PART):
        k = slice(i, i + PART)
        a, b, c = m.first_hit_backward(V, S[k].contiguous(), E[k].contiguous(), tri[k].contiguous(), gt[k].contiguous(),
                                       guv[k].contiguous(), gp[k].contiguous())
        assert torch.equal(b, dS[k]) and torch.equal(c, dE[k])
        total += a.double()
        size += a.double().abs()
    assert float(size.max()) > 0
    assert torch.all((dV.double() - total).abs() <= 2.0 ** -23 * (size + total.abs()))
    m.close()
