"""A captured call over instances of 64 loops or fewer is one chain of kernels on
the capturing stream: groups in shared launches, members with a variant of
their own (as branches whose streams wait for each other both ways, these
crashed the runtime at the end of the capture), and one instance alone in its
size; every replay equals the instances' own calls bit for bit, after eager
work between the replays."""
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("prec,variant", [(0, 0), (1, 1), (2, 0), (2, 1)])
def test_captured_chain(prec, variant):
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device")
    from paper_2503_18479_amd import LOSS_RATIO, Geometry, Plan, capture_loss_and_grad_many
    shapes = [(4, 4, 2, 20, 3), (5, 5, 1, 25, 2), (6, 6, 2, 18, 1), (7, 7, 1, 22, 4), (8, 8, 13, 16, 2)]
    if variant == 1:
        shapes = shapes[:3]  # 36 loops alone in its size
    wls = [W.small_array(nx, ny, batch=b, grid=g, n_freq=f, seed=60 + i)
           for i, (nx, ny, b, g, f) in enumerate(shapes)]
    t = lambda a: torch.tensor(a, device="cuda:0")
    plans = [Plan(Geometry.from_workload(w.geom), t(w.pts), w.bext_z) for w in wls]
    for p in plans[:2]:
        p.set_variant(prec, variant)
    Cs, Os = [t(w.C) for w in wls], [t(w.omega) for w in wls]
    Ts = [1.0 + 0.5 * t(w.target) / float(w.target.max()) for w in wls]
    graph, outs = capture_loss_and_grad_many(plans, Cs, Os, Ts, LOSS_RATIO, prec)
    for rep in range(3):
        for C in Cs:
            C.mul_(1.0 + 0.02 * (rep + 1))
        ref = [p.loss_and_grad(C, o, T, LOSS_RATIO, prec) for p, C, o, T in zip(plans, Cs, Os, Ts)]
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for out, r in zip(outs, ref):
            assert all(torch.equal(a, b) for a, b in zip(out, r)), rep
