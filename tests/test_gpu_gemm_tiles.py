"""The two-pass contraction above 64 loops at the edges of its tiles, against the
FP64 oracle: point and loop counts that are no multiple of the row tile, item
counts that are no multiple of eight (the share of each XCD), several chunks
of points, in each precision."""
import numpy as np
import pytest

import oracle as O
import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

TOL = {0: 1e-9, 1: 1e-4, 2: 1e-4}


@pytest.mark.parametrize("prec", [0, 1, 2])
#                                    loops, points:  blocks of 64
@pytest.mark.parametrize("nx,ny,grid,batch,nf", [(13, 5, 9, 64, 2),    # 2, 2
                                                 (12, 11, 14, 33, 4),  # 3, 4
                                                 (17, 16, 41, 65, 2)])  # 5, 27
def test_two_pass_contraction(nx, ny, grid, batch, nf, prec):
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device")
    from paper_2503_18479_amd import Geometry, Plan
    dev = torch.device("cuda:0")
    print(f"[gemm tiles] {nx * ny} loops, {grid * grid} points, {batch * nf} systems, prec={prec}", flush=True)
    wl = W.small_array(nx, ny, batch=batch, grid=grid, n_freq=nf, seed=nx)
    g = wl.geom
    t = lambda a: torch.tensor(a, device=dev)
    plan = Plan(Geometry.from_workload(g), t(wl.pts), wl.bext_z)
    loss, grad, st = plan.loss_and_grad(t(wl.C), t(wl.omega), t(wl.target), precision=prec)
    assert int(st.abs().sum()) == 0
    ok = [0, batch // 2, batch - 1]
    G = O.field_matrix(g.verts, g.seg_off, wl.pts)
    M = O.inductance_matrix_lattice(g.verts, g.seg_off, g.wire_a, nx, ny)
    Phi = O.flux(g.verts, g.seg_off, wl.bext_z)
    Lr = O.evaluate(G, M, g.R, Phi, wl.C[ok], wl.omega, wl.target)[2]
    gr = O.grad_adjoint(G, M, g.R, Phi, wl.C[ok], wl.omega, wl.target)
    loss, grad = loss.cpu().numpy()[ok], grad.cpu().numpy()[ok]
    assert np.all(np.abs(loss - Lr) <= TOL[prec] * np.abs(Lr))
    assert np.all(np.linalg.norm(grad - gr, axis=1) <= TOL[prec] * np.linalg.norm(gr, axis=1))
