"""33 to 64 loops at the edge between the launches of few systems (a workgroup
per system, the inverse of L recorded, up to 48) and of many (a wave per
system): currents, loss and gradient and the field's backward pass from the
record, against the FP64 oracle, with systems that need the pivoted
elimination among the others."""
import numpy as np
import pytest

import oracle as O
import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("nx,ny,batch,nf", [(11, 3, 1, 1), (11, 3, 3, 2), (7, 7, 48, 1), (8, 8, 17, 3),
                                            (8, 6, 16, 3), (8, 8, 1, 5), (13, 4, 49, 1)])
def test_few_systems(nx, ny, batch, nf):
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device")
    from paper_2503_18479_amd import Geometry, Plan, cosim_field
    dev = torch.device("cuda:0")
    print(f"[few systems] {nx * ny} loops, {batch} x {nf} systems", flush=True)
    wl = W.small_array(nx, ny, batch=batch, grid=9, n_freq=nf, seed=nx + batch)
    g, w, C = wl.geom, wl.omega, wl.C.copy()
    t = lambda a: torch.tensor(a, device=dev)
    plan = Plan(Geometry.from_workload(g), t(wl.pts), wl.bext_z, precisions=["fp64"])
    M = O.inductance_matrix_fast(g.verts, g.seg_off, g.wire_a)
    G = O.field_matrix(g.verts, g.seg_off, wl.pts)
    Phi = O.flux(g.verts, g.seg_off, wl.bext_z)
    bad = []
    if batch > 1:
        bad, C[1, -1] = [1], 0.0
        C[2 % batch, 0] = 1.0 / (w[0] ** 2 * M[0, 0])  # loop 0 at resonance: a small pivot
    ok = [i for i in (0, 2, batch // 2, batch - 1) if i < batch and i not in bad]
    ok = sorted(set(ok))
    I, st = plan.solve(t(C), t(w))
    assert (st[bad] == 1).all() and bool(torch.isnan(torch.view_as_real(I[bad])).all())
    assert int(st.sum()) == len(bad) * nf
    Ir = O.currents(M, g.R, Phi, C[ok], w)
    err = np.linalg.norm(I.cpu().numpy()[ok] - Ir, axis=2) / np.linalg.norm(Ir, axis=2)
    assert err.max() <= 1e-9
    loss, grad, st = plan.loss_and_grad(t(C), t(w), t(wl.target), 0, 0)
    Lr = O.evaluate(G, M, g.R, Phi, C[ok], w, wl.target)[2]
    gr = O.grad_adjoint(G, M, g.R, Phi, C[ok], w, wl.target)
    loss, grad = loss.cpu().numpy(), grad.cpu().numpy()
    assert np.isnan(loss[bad]).all() and np.isnan(grad[bad]).all()
    assert np.all(np.abs(loss[ok] - Lr) <= 1e-9 * np.abs(Lr))
    assert np.all(np.linalg.norm(grad[ok] - gr, axis=1) <= 1e-9 * np.linalg.norm(gr, axis=1))
    # the field's backward pass replays the record of its forward pass
    Cf = C.copy()
    Cf[bad] = wl.C[bad]
    x = t(Cf).requires_grad_(True)
    B = cosim_field(x, plan, t(w), "fp64")
    T = t(wl.target)
    # the same loss in torch operations
    (((B.abs() - T) ** 2).sum() / (B.shape[1] * B.shape[2])).backward()
    gb, scale = x.grad.cpu().numpy()[ok], np.linalg.norm(gr, axis=1)
    k = np.sum(gb * gr) / np.sum(gr * gr)  # the two losses differ by a constant factor
    assert np.all(np.linalg.norm(gb - k * gr, axis=1) <= 1e-9 * abs(k) * scale)


def test_group_of_few_and_many_matches_single_calls():
    """A grouped call whose members of 33 to 64 loops lie on both sides of the
    line gives each the bits of its own call, capacitance by capacitance."""
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device")
    from paper_2503_18479_amd import Geometry, Plan, loss_and_grad_many
    dev = torch.device("cuda:0")
    wls = [W.small_array(nx, ny, batch=b, grid=12, n_freq=f, seed=b)
           for nx, ny, b, f in ((8, 8, 49, 1), (8, 8, 5, 2), (7, 6, 48, 1), (7, 7, 25, 2), (11, 3, 1, 1))]
    t = lambda a: torch.tensor(a, device=dev)
    plans = [Plan(Geometry.from_workload(w.geom), t(w.pts), w.bext_z) for w in wls]
    Cs, Os, Ts = [t(w.C) for w in wls], [t(w.omega) for w in wls], [t(w.target) for w in wls]
    Cs[0][3, 1] = 0.0  # an invalid configuration on either side
    Cs[1][2, 0] = 0.0
    for prec in (0, 2):
        print(f"[few and many] prec={prec}", flush=True)
        outs = loss_and_grad_many(plans, Cs, Os, Ts, precision=prec)
        for p, C, om, T, out in zip(plans, Cs, Os, Ts, outs):
            for a, b in zip(out, p.loss_and_grad(C, om, T, precision=prec)):
                assert torch.equal(torch.nan_to_num(a.double()), torch.nan_to_num(b.double()))
                assert torch.equal(torch.isnan(a.double()), torch.isnan(b.double()))
    assert int(outs[0][2].sum()) == 1 and int(outs[1][2].sum()) == 2
