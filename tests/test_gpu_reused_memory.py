"""A plan destroyed while its work is still enqueued on another stream, and a
plan built at once on its memory: the old work reads the old operators."""
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def test_new_plan_waits_for_the_old_ones_work():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device")
    from paper_2503_18479_amd import Geometry, Plan
    dev = torch.device("cuda:0")
    t = lambda a: torch.tensor(a, device=dev)
    wl = W.small_array(8, 8, batch=64, grid=128, n_freq=2, seed=1)
    geo, pts = Geometry.from_workload(wl.geom), t(wl.pts)
    I, _ = Plan(geo, pts, wl.bext_z).solve(t(wl.C), t(wl.omega))
    keep = Plan(geo, pts, wl.bext_z)
    want = keep.field(I)
    shifted = pts + 0.01
    other = Plan(geo, shifted, wl.bext_z).G()
    side = torch.cuda.Stream()
    for rep in range(3):
        old = Plan(geo, pts, wl.bext_z)  # no workspace: nothing else waits when it goes
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            got = [old.field(I) for _ in range(8)]
        del old
        new = Plan(geo, shifted, wl.bext_z)  # before anything is waited for
        assert torch.equal(new.G(), other), rep
        torch.cuda.synchronize()
        assert all(torch.equal(g, want) for g in got), rep
        del new
