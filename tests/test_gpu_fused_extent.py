"""The FP64 and FP32 fused contraction at the loop counts where its extent (the
columns and adjoint row blocks it leaves out) changes, against the FP64 oracle
in every loss mode; one grouped call per precision with two extents against
single calls; and a field that is zero everywhere."""
import numpy as np
import pytest

import oracle as O
import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

TOL = {0: 1e-9, 1: 1e-5}


def _setup(nx, ny, seed, bext=None):
    from paper_2503_18479_amd import Geometry, Plan
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device")
    dev = torch.device("cuda:0")
    wl = W.small_array(nx, ny, batch=23, grid=11, n_freq=3, seed=seed)  # 121 points, 69 systems
    plan = Plan(Geometry.from_workload(wl.geom), torch.tensor(wl.pts, device=dev),
                wl.bext_z if bext is None else bext, precisions=["fp64", "fp32"])
    t = lambda a: torch.tensor(a, device=dev)
    return wl, plan, t(wl.C), t(wl.omega), t(wl.target)


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("nx,ny", [(8, 1), (3, 3), (4, 4), (17, 1), (8, 4), (11, 3), (8, 6), (7, 7)])
def test_extents_match_oracle(nx, ny, prec):
    wl, plan, C, om, T = _setup(nx, ny, 10 * nx + ny)
    g = wl.geom
    print(f"[fused extent] {g.n} loops prec={prec}", flush=True)
    G = O.field_matrix(g.verts, g.seg_off, wl.pts)
    M = O.inductance_matrix_fast(g.verts, g.seg_off, g.wire_a)
    Phi = O.flux(g.verts, g.seg_off, wl.bext_z)
    for mode in (0, 1, 2):
        Tm = wl.target if mode < 2 else 1.0 + wl.target / wl.bext_z
        loss, grad, st = plan.loss_and_grad(C, om, torch.tensor(Tm, device=C.device), mode, prec)
        Lr = O.evaluate(G, M, g.R, Phi, wl.C, wl.omega, Tm, mode, wl.bext_z)[2]
        gr = O.grad_adjoint(G, M, g.R, Phi, wl.C, wl.omega, Tm, mode, wl.bext_z)
        assert int(st.abs().sum()) == 0
        assert np.all(np.abs(loss.cpu().numpy() - Lr) <= TOL[prec] * np.abs(Lr)), mode
        e = np.linalg.norm(grad.cpu().numpy() - gr, axis=1) / np.linalg.norm(gr, axis=1)
        assert e.max() <= TOL[prec], (mode, e.max())


@pytest.mark.parametrize("prec", [0, 1])
def test_grouped_extents_equal_single_calls(prec):
    from paper_2503_18479_amd import loss_and_grad_many
    cases = [_setup(8, 1, 1), _setup(3, 3, 2), _setup(8, 6, 3), _setup(8, 8, 4)]
    outs = loss_and_grad_many([c[1] for c in cases], [c[2] for c in cases], [c[3] for c in cases],
                              [c[4] for c in cases], precision=prec)
    for (_, plan, C, om, T), (l, g, s) in zip(cases, outs):
        l1, g1, s1 = plan.loss_and_grad(C, om, T, precision=prec)
        assert torch.equal(l, l1) and torch.equal(g, g1) and torch.equal(s, s1)


def test_zero_field():
    """No incident field: every current and field value is zero, the loss is
    the mean of T^2 (exact up to the rounding of its sum) and the gradient 0."""
    wl, plan, C, om, T = _setup(3, 3, 5, bext=0.0)
    for prec in (0, 1):
        loss, grad, st = plan.loss_and_grad(C, om, T, 0, prec)
        ref = float(np.mean(wl.target ** 2))
        assert np.all(np.abs(loss.cpu().numpy() - ref) <= (1e-12, 1e-6)[prec] * ref)
        assert not grad.cpu().numpy().any()
