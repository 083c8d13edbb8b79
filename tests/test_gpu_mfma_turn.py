"""BF16X3 loss and gradient above 64 loops with few systems, where the adjoint's
operands are turned in LDS from the forward's, at loop counts around the
16-loop tiles, 32-loop steps and 64-loop waves, against the FP64 oracle; the
loss of a call without gradient (which turns nothing) must be the same bits."""
import numpy as np
import pytest

import oracle as O
import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("nx,ny", [(13, 5), (16, 5), (27, 3), (16, 6), (97, 1), (16, 8), (43, 3),
                                   (12, 12), (23, 7), (16, 16), (29, 9), (32, 16)])
def test_turned_operands(nx, ny):
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device")
    from paper_2503_18479_amd import Geometry, Plan
    dev = torch.device("cuda:0")
    wl = W.small_array(nx, ny, batch=5, grid=9, n_freq=4, seed=nx)  # 81 points, 20 systems
    g = wl.geom
    print(f"[turn] {g.n} loops", flush=True)
    plan = Plan(Geometry.from_workload(g), torch.tensor(wl.pts, device=dev), wl.bext_z)
    a = [torch.tensor(x, device=dev) for x in (wl.C, wl.omega, wl.target)]
    loss, grad, st = plan.loss_and_grad(*a, precision="bf16x3")
    only = plan.loss_and_grad(*a, precision="bf16x3", grad=False)[0]
    assert torch.equal(loss, only) and int(st.abs().sum()) == 0
    G = O.field_matrix(g.verts, g.seg_off, wl.pts)
    M = O.inductance_matrix_lattice(g.verts, g.seg_off, g.wire_a, nx, ny)
    Phi = O.flux(g.verts, g.seg_off, wl.bext_z)
    Lr = O.evaluate(G, M, g.R, Phi, wl.C, wl.omega, wl.target)[2]
    gr = O.grad_adjoint(G, M, g.R, Phi, wl.C, wl.omega, wl.target)
    assert np.all(np.abs(loss.cpu().numpy() - Lr) <= 3e-3 * np.abs(Lr))
    e = np.linalg.norm(grad.cpu().numpy() - gr, axis=1) / np.linalg.norm(gr, axis=1)
    assert e.max() <= 3e-3, e.max()
