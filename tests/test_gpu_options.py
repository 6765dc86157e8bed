"""Launch options: what rsi_get_opts reports can be set again without changing
the launch, and the defaults can be set back.  The thresholds in force show
in the number of refills of the counting walk."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2209_02878_amd import rsi
from paper_2209_02878_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _t(a, dtype=torch.float32):
    return torch.as_tensor(np.ascontiguousarray(a)).to(device="cuda", dtype=dtype).contiguous()


@pytest.mark.parametrize("mode", ["count", "all"])
def test_round_trip(mode):
    V, T = wl.noisy_sphere(30, 4, 0.3)
    S, E = wl.segments_in_box(np.random.default_rng(9), V.min(0), V.max(0), 2_000_000, scale=1.5)
    mesh = rsi.Mesh(_t(V), _t(T, torch.int32))
    S, E = _t(S), _t(E)

    def refills():
        mesh.set_counting(True)
        mesh.query(S, E, mode, capacity=4)
        torch.cuda.synchronize()
        n = mesh.counters()["wave_refills"]
        mesh.set_counting(False)
        return n

    opts, base = mesh.opts(), refills()
    assert (opts["block_size"], opts["defer_lanes"], opts["refill_lanes"]) == (128, 32, 32)
    mesh.set_opts(**opts)
    assert mesh.opts() == opts
    assert abs(refills() - base) < 0.04 * base
    mesh.set_opts(block_size=64, defer_lanes=16, refill_lanes=56)
    assert refills() < 0.8 * base
    mesh.set_opts(**opts)
    assert mesh.opts() == opts
    assert abs(refills() - base) < 0.04 * base
    mesh.close()
