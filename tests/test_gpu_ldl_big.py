"""The blocked LDL^T above 64 loops at the edges of its blocking, against the
FP64 oracle: one row past a block of 64, whole blocks, and the block counts
where the trailing update after four block rows starts (6), ends (9) and runs
twice (10); with and without the complex64 record, with one invalid system."""
import numpy as np
import pytest

import oracle as O
import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

#                 loops: blocks
SHAPES = [(13, 5), (16, 8), (16, 20), (19, 19), (23, 23), (25, 25)]


@pytest.mark.parametrize("refine", [False, True])
@pytest.mark.parametrize("nx,ny", SHAPES)
def test_blocked_ldl_matches_oracle(nx, ny, refine):
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device")
    from paper_2503_18479_amd import Geometry, Plan
    dev = torch.device("cuda:0")
    wl = W.small_array(nx, ny, batch=3, grid=8, n_freq=3, seed=nx)
    g = wl.geom
    print(f"[ldl blocks] {g.n} loops refine={refine}", flush=True)
    C = wl.C.copy()
    C[1, 5] = 0.0  # configuration 1 is invalid at every frequency
    plan = Plan(Geometry.from_workload(g), torch.tensor(wl.pts, device=dev), wl.bext_z)
    if refine:
        plan.set_refinement(True)
    Cd, om = torch.tensor(C, device=dev), torch.tensor(wl.omega, device=dev)
    I, st = plan.solve(Cd, om)
    G = O.field_matrix(g.verts, g.seg_off, wl.pts)
    M = O.inductance_matrix_lattice(g.verts, g.seg_off, g.wire_a, nx, ny)
    Phi = O.flux(g.verts, g.seg_off, wl.bext_z)
    ok = [0, 2]
    Ir = O.currents(M, g.R, Phi, C[ok], wl.omega)
    I = I.cpu().numpy()
    assert np.isnan(I[1]).all() and int(st[1].min()) == 1 and int(st[ok].abs().sum()) == 0
    assert np.linalg.norm(I[ok] - Ir) <= 1e-9 * np.linalg.norm(Ir)
    loss, grad, st = plan.loss_and_grad(Cd, om, torch.tensor(wl.target, device=dev), precision=0)
    Lr = O.evaluate(G, M, g.R, Phi, C[ok], wl.omega, wl.target)[2]
    gr = O.grad_adjoint(G, M, g.R, Phi, C[ok], wl.omega, wl.target)
    loss, grad = loss.cpu().numpy(), grad.cpu().numpy()
    assert np.isnan(loss[1]) and np.isnan(grad[1]).all()
    assert np.all(np.abs(loss[ok] - Lr) <= 1e-9 * np.abs(Lr))
    assert np.all(np.linalg.norm(grad[ok] - gr, axis=1) <= 1e-9 * np.linalg.norm(gr, axis=1))
