"""Eager grouped calls with instances above 64 loops: three of 81 loops
(different batches, frequency counts and points), two of 144 and two small
ones, factored and solved together; every result equals the instance's own
call bit for bit, in three precisions and every loss mode, with and without
gradients."""
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def test_grouped_large_instances_eager():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device")
    from paper_2503_18479_amd import LOSS_COMPLEX, LOSS_MAG, LOSS_RATIO, Geometry, Plan, loss_and_grad_many
    wls = [W.small_array(nx, ny, batch=b, grid=g, n_freq=f, seed=41 + i) for i, (nx, ny, b, g, f) in
           enumerate([(9, 9, 2, 30, 3), (9, 9, 1, 45, 1), (12, 12, 2, 20, 2), (3, 2, 3, 16, 2),
                      (9, 9, 3, 24, 2), (12, 12, 1, 28, 3), (5, 5, 2, 18, 1)])]
    t = lambda a: torch.tensor(a, device="cuda:0")
    plans = [Plan(Geometry.from_workload(w.geom), t(w.pts), w.bext_z) for w in wls]
    Cs, Os, Ts = [t(w.C) for w in wls], [t(w.omega) for w in wls], [t(w.target) for w in wls]
    Rs = [1.0 + 0.5 * T / T.max() for T in Ts]
    for prec, mode, grad in [(0, LOSS_MAG, True), (1, LOSS_MAG, True), (2, LOSS_MAG, True),
                             (2, LOSS_COMPLEX, True), (2, LOSS_COMPLEX, False), (2, LOSS_RATIO, True),
                             (2, LOSS_RATIO, False)]:
        print(f"[grouped large] prec={prec} mode={mode} grad={grad}", flush=True)
        tg = Rs if mode == LOSS_RATIO else Ts
        many = loss_and_grad_many(plans, Cs, Os, tg, loss_mode=mode, precision=prec, grad=grad)
        for pl, C, o, T, (l, g, s) in zip(plans, Cs, Os, tg, many):
            l1, g1, s1 = pl.loss_and_grad(C, o, T, loss_mode=mode, precision=prec, grad=grad)
            assert torch.equal(l, l1) and torch.equal(s, s1) and int(s.abs().sum()) == 0
            assert (g is None) == (not grad) and (g is None or torch.equal(g, g1))
