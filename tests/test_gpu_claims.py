"""Work items handed out: where one chunk a wave covers every item the waves'
items are fixed, else they are claimed from eight ranges.  Around the change
(it lies at 64 items per resident wave), at counts that leave ranges and
workgroups empty, and with a chunk set by the caller, every segment is walked
once (work counters) and answers as in a launch of another size."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2209_02878_amd import rsi
from paper_2209_02878_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _t(a, dtype=torch.float32):
    return torch.as_tensor(np.ascontiguousarray(a)).to(device="cuda", dtype=dtype).contiguous()


@pytest.mark.parametrize("branching", [2, 4])
@pytest.mark.parametrize("chunk", [0, 64, 4096])
def test_every_segment_once(branching, chunk):
    V, T = wl.noisy_sphere(9, 4, 0.3)
    S, E = wl.segments_in_box(np.random.default_rng(2), V.min(0), V.max(0), 600_011, scale=1.5)
    S, E = _t(S), _t(E)
    mesh = rsi.Mesh(_t(V), _t(T, torch.int32), branching=branching, chunk=chunk)
    want = mesh.query(S, E, "first|count")
    waves = torch.cuda.get_device_properties(0).multi_processor_count * 4
    sizes = [1, 3, 7, 9, 63, 186, 1_537, 98_303, 98_305, 600_011]
    sizes += [64 * waves * k + d for k in range(4, 9) for d in (-1, 0, 1) if 64 * waves * k < 600_000]
    for n in sizes:
        got = mesh.query(S[:n].clone(), E[:n].clone(), "first|count")
        for k in got:
            assert torch.equal(got[k], want[k][:n]), (n, k)
    mesh.set_counting(True)
    for n in sizes:
        mesh.query(S[:n].clone(), E[:n].clone(), "count")
        torch.cuda.synchronize()
        assert mesh.counters()["segments"] == n, n
    mesh.close()
