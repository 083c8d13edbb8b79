"""33 to 64 loops on both sides of the line between a workgroup and a wave per
system (12 systems of a plan): currents, loss, gradient and the field's
backward pass, which replays the record, against the FP64 oracle without a
free factor; and members on either side in one grouped call, which get the
bits of their own calls."""
import numpy as np
import pytest

import oracle as O
import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("nx,ny,batch,nf", [(11, 3, 12, 1), (11, 3, 13, 1), (7, 7, 4, 3), (8, 8, 13, 1),
                                            (8, 8, 3, 4), (8, 6, 7, 2), (8, 8, 1, 1)])
def test_either_side_of_the_line(nx, ny, batch, nf):
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device")
    from paper_2503_18479_amd import Geometry, Plan, cosim_field
    print(f"[line] {nx * ny} loops, {batch} x {nf} systems", flush=True)
    wl = W.small_array(nx, ny, batch=batch, grid=9, n_freq=nf, seed=nx + batch)
    g, w, C = wl.geom, wl.omega, wl.C
    t = lambda a: torch.tensor(a, device="cuda:0")
    plan = Plan(Geometry.from_workload(g), t(wl.pts), wl.bext_z, precisions=["fp64"])
    M = O.inductance_matrix_fast(g.verts, g.seg_off, g.wire_a)
    G = O.field_matrix(g.verts, g.seg_off, wl.pts)
    Phi = O.flux(g.verts, g.seg_off, wl.bext_z)
    I, st = plan.solve(t(C), t(w))
    Ir = O.currents(M, g.R, Phi, C, w)
    assert int(st.sum()) == 0
    err = np.linalg.norm(I.cpu().numpy() - Ir, axis=2) / np.linalg.norm(Ir, axis=2)
    assert err.max() <= 1e-9
    loss, grad, _ = plan.loss_and_grad(t(C), t(w), t(wl.target), 0, 0)
    Lr = O.evaluate(G, M, g.R, Phi, C, w, wl.target)[2]
    gr = O.grad_adjoint(G, M, g.R, Phi, C, w, wl.target)
    norm = np.linalg.norm(gr, axis=1)
    assert np.all(np.abs(loss.cpu().numpy() - Lr) <= 1e-9 * np.abs(Lr))
    assert np.all(np.linalg.norm(grad.cpu().numpy() - gr, axis=1) <= 1e-9 * norm)
    x = t(C).requires_grad_(True)
    B = cosim_field(x, plan, t(w), "fp64")
    before = plan.factorisations()
    # the mean of (|B| - T)^2 over frequencies and points, summed over the batch
    (((B.abs() - t(wl.target)) ** 2).sum() / (B.shape[1] * B.shape[2])).backward()
    assert plan.factorisations() == before  # the record was replayed
    assert np.all(np.linalg.norm(x.grad.cpu().numpy() - gr, axis=1) <= 1e-9 * norm)


def test_group_across_the_line_matches_single_calls():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device")
    from paper_2503_18479_amd import Geometry, Plan, loss_and_grad_many
    wls = [W.small_array(nx, ny, batch=b, grid=12, n_freq=f, seed=b)
           for nx, ny, b, f in ((8, 8, 13, 1), (8, 8, 6, 2), (7, 6, 12, 1), (7, 7, 7, 2), (11, 3, 1, 1))]
    t = lambda a: torch.tensor(a, device="cuda:0")
    plans = [Plan(Geometry.from_workload(w.geom), t(w.pts), w.bext_z) for w in wls]
    Cs, Os, Ts = [t(w.C) for w in wls], [t(w.omega) for w in wls], [t(w.target) for w in wls]
    for prec in (0, 1, 2):
        outs = loss_and_grad_many(plans, Cs, Os, Ts, precision=prec)
        for p, C, om, T, out in zip(plans, Cs, Os, Ts, outs):
            for a, b in zip(out, p.loss_and_grad(C, om, T, precision=prec)):
                assert torch.equal(a, b)


@pytest.mark.parametrize("batch", [2, 10, 40])
def test_status_of_the_record(batch):
    """The replay starts from the recorded status: an invalid configuration and
    one that needs the pivoted elimination, on either side of the line."""
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device")
    from paper_2503_18479_amd import Geometry, Plan
    wl = W.small_array(8, 8, batch=batch, grid=9, n_freq=4, seed=batch)
    t = lambda a: torch.tensor(a, device="cuda:0")
    plan = Plan(Geometry.from_workload(wl.geom), t(wl.pts), wl.bext_z)
    C = wl.C.copy()
    C[0, 0] = 1.0 / (wl.omega[0] ** 2 * plan.M()[0, 0])  # a small pivot
    C[1, 7] = 0.0
    C[-1, 3] *= -1.0 if batch > 2 else 1.0
    I, st = plan.solve(t(C), t(wl.omega))
    want = torch.zeros((batch, 4), dtype=torch.int32, device="cuda:0")
    want[1] = 1
    if batch > 2:
        want[-1] = 8
    assert torch.equal(st, want)
    gB = torch.ones((batch, 4, plan.P), dtype=torch.complex128, device="cuda:0")
    gC, st2 = plan.field_backward(t(C), t(wl.omega), I, gB, reuse=True)
    assert torch.equal(st2, want)
    assert bool(torch.isnan(gC[1]).all()) and not bool(torch.isnan(gC[0]).any())
    ref, st3 = plan.field_backward(t(C), t(wl.omega), I, gB)
    ok = [b for b in range(batch) if b != 1]
    assert torch.equal(st3, want)
    assert float((gC[ok] - ref[ok]).norm()) <= 1e-9 * float(ref[ok].norm())
