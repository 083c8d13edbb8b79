"""Plans built and destroyed while another thread captures a graph in a mode
that allows it (thread-local or relaxed): neither the capture nor the plans
suffer, also when a plan takes over a destroyed one's memory."""
import threading

import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("mode", ["thread_local", "relaxed"])
def test_plans_beside_a_capture(mode):
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device")
    from paper_2503_18479_amd import Geometry, Plan
    dev = torch.device("cuda:0")
    t = lambda a: torch.tensor(a, device=dev)
    wl = W.small_array(4, 4, batch=8, grid=32, n_freq=1, seed=0)
    geo, pts = Geometry.from_workload(wl.geom), t(wl.pts)
    C, om, T = t(wl.C), t(wl.omega), t(wl.target)
    plan = Plan(geo, pts, wl.bext_z)
    plan.reserve(8, 1)
    G = plan.G()
    out = (torch.empty(8, dtype=torch.float64, device=dev),
           torch.empty((8, 16), dtype=torch.float64, device=dev),
           torch.empty((8, 1), dtype=torch.int32, device=dev))
    plan.loss_and_grad(C, om, T, out=out)
    want = [o.clone() for o in out]
    torch.cuda.synchronize()
    old = Plan(geo, pts, wl.bext_z)
    del old  # memory for the other thread's plans to take over
    go, done, other = threading.Event(), threading.Event(), []

    def build():
        torch.cuda.set_device(dev)
        with torch.cuda.stream(torch.cuda.Stream()):
            go.wait(30)
            try:
                for _ in range(3):
                    other.append(Plan(geo, pts, wl.bext_z).M().sum())
            except Exception as e:  # reported below
                other.append(e)
        done.set()

    th = threading.Thread(target=build)
    th.start()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, capture_error_mode=mode):
        go.set()
        assert done.wait(30)
        plan.loss_and_grad(C, om, T, out=out)
    th.join()
    assert other == [plan.M().sum()] * 3
    for _ in range(3):
        for o in out:
            o.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(out, want))
        assert torch.equal(Plan(geo, pts, wl.bext_z).G(), G)  # eager work between the replays
