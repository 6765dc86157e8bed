"""More than 2^26 triangles, whose records lie past a 32-bit byte offset: the
four-way walk is used there too (it tests more than two boxes per visit, the
binary one exactly two) and gives the binary walk's answers, at the far end
of the records among others."""
import pytest

torch = pytest.importorskip("torch")

from paper_2209_02878_amd import rsi

pytestmark = pytest.mark.gpu


def test_four_way_walk_past_2_26_triangles():
    m = 5_793  # cells per side
    n = m + 1
    gen = torch.Generator(device="cuda").manual_seed(4)
    g = torch.arange(n, device="cuda", dtype=torch.float32) / m
    z = 0.01 * torch.sin(40 * g)[None, :] * torch.cos(30 * g)[:, None]
    V = torch.stack([g.repeat(n), g.repeat_interleave(n), z.reshape(-1)], 1).contiguous()
    i = torch.arange(m, device="cuda", dtype=torch.int32)
    v = (i[:, None] * n + i[None, :]).reshape(-1)
    T = torch.stack([v, v + 1, v + n + 1, v, v + n + 1, v + n], 1).reshape(-1, 3).contiguous()
    del v
    assert T.shape[0] > 1 << 26
    mesh = rsi.Mesh(V, T)
    for count in (3_000, 400_000):  # shared walks without, and walks with, the copy of the top records
        xy = torch.rand(count, 2, device="cuda", generator=gen)
        xy[::2] = 1 - 0.002 * xy[::2]  # the last triangles in Morton order
        d = 0.003 * (torch.rand(count, 2, device="cuda", generator=gen) - 0.5)
        S = torch.cat([xy, torch.full_like(xy[:, :1], 0.02)], 1).contiguous()
        E = torch.cat([xy + d, torch.full_like(xy[:, :1], -0.02)], 1).contiguous()
        out = {}
        for width in (4, 2):
            mesh.set_opts(branching=width)
            out[width] = mesh.query(S, E, "first|count")
            mesh.set_counting(True)
            mesh.query(S, E, "count")
            torch.cuda.synchronize()
            c = mesh.counters()
            mesh.set_counting(False)
            assert (c["box_tests"] > 2 * c["node_visits"]) == (width == 4), c
        assert int(out[4]["count"].sum()) > 0.9 * count
        for k in out[2]:
            assert torch.equal(out[4][k], out[2][k]), k
    mesh.set_opts(branching=4)
    # the same mesh behind a small one in a batch
    batch = rsi.Batch([(V[:n + 2].clone(), T[:2].clone()), (V, T)])
    got = batch.query([(S[:5], E[:5]), (S, E)], "first")[1]
    want = mesh.query(S, E, "first")
    for k in want:
        assert torch.equal(got[k], want[k]), k
    batch.close()
    mesh.close()
