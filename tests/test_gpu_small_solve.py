"""The forward solve of 64 loops or fewer at the edges of its launch rules: one
wave and one launch up to 32 loops (panels of 8), factorisation and
substitution in one launch up to 2,048 systems of 33 to 64 loops, and the
fallback's scan over blocks of 32 systems; and the final sums that the adjoint
replay forms for one frequency."""
import numpy as np
import pytest

import oracle as O
import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _case(nx, ny, batch, nf, seed, R=0.3):
    from paper_2503_18479_amd import Geometry, Plan
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device")
    dev = torch.device("cuda:0")
    wl = W.small_array(nx, ny, batch=batch, grid=9, n_freq=nf, seed=seed)
    g = wl.geom
    plan = Plan(Geometry(g.verts, g.seg_off, g.wire_a, R), torch.tensor(wl.pts, device=dev),
                wl.bext_z, precisions=["fp64"])
    t = lambda a: torch.tensor(a, device=dev)
    M = O.inductance_matrix_fast(g.verts, g.seg_off, g.wire_a)
    Phi = O.flux(g.verts, g.seg_off, wl.bext_z)
    return wl, plan, t, M, Phi, np.full(g.n, R)


@pytest.mark.parametrize("nx,ny,batch", [(1, 1, 70), (7, 1, 70), (8, 1, 70), (3, 3, 70), (31, 1, 70),
                                         (8, 4, 70), (11, 3, 70), (8, 8, 70), (8, 8, 690), (31, 1, 690)])
def test_forward_solve_and_fallback_scan(nx, ny, batch):
    """Invalid systems at the edges of the scan, a system with a tiny pivot
    (its first loop at resonance), the rest against the oracle."""
    wl, plan, t, M, Phi, R = _case(nx, ny, batch, 3, nx + ny, R=1e-6)
    print(f"[small solve] {nx * ny} loops, {batch} configurations", flush=True)
    w = wl.omega
    C = wl.C.copy()
    bad = [0, 10, batch - 1]       # systems 0-2, 30-32 (across two scan blocks) and the last three
    C[bad, -1] = 0.0
    C[5, 0] = 1.0 / (w[1] ** 2 * M[0, 0])  # zero reactance of loop 0 at frequency 1
    I, st = plan.solve(t(C), t(w))
    I, st = I.cpu().numpy(), st.cpu().numpy()
    ok = [i for i in (1, 5, 9, 11, 33, batch - 2) if i not in bad]
    assert (st[bad] == 1).all() and np.isnan(I[bad]).all()
    rest = np.delete(st, bad, axis=0)
    assert (rest == 0).all()
    ref = O.currents(M, R, Phi, C[ok], w)
    err = np.linalg.norm(I[ok] - ref, axis=2) / np.linalg.norm(ref, axis=2)
    # nearly lossless loops: the condition number grows as |Z_kk| / R
    assert err.max() < 1e-9 * max(1.0, np.abs(w[0] * M[0, 0]) / R[0] * 1e-4), err.max()


@pytest.mark.parametrize("nx,ny", [(1, 1), (5, 5), (8, 8)])
def test_single_frequency_sums(nx, ny):
    wl, plan, t, M, Phi, R = _case(nx, ny, 67, 1, 3)
    C, om, T = t(wl.C), t(wl.omega), t(wl.target)
    loss, grad, st = plan.loss_and_grad(C, om, T, 0, 0)
    only, none, _ = plan.loss_and_grad(C, om, T, 0, 0, grad=False)  # the sums of a separate launch
    assert none is None and torch.equal(loss, only)
    G = O.field_matrix(wl.geom.verts, wl.geom.seg_off, wl.pts)
    Lr = O.evaluate(G, M, R, Phi, wl.C, wl.omega, wl.target)[2]
    gr = O.grad_adjoint(G, M, R, Phi, wl.C, wl.omega, wl.target)
    assert np.all(np.abs(loss.cpu().numpy() - Lr) <= 1e-9 * np.abs(Lr))
    g = grad.cpu().numpy()
    assert np.all(np.linalg.norm(g - gr, axis=1) <= 1e-9 * np.linalg.norm(gr, axis=1))
    assert int(st.abs().sum()) == 0
