"""Loops without a capacitor (C = +inf) have gradient 0: with one frequency, too,
it is the +0 that the sum over frequencies gives, so that grouped calls and
single ones agree to the last bit."""
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("shape", [(4, 4), (8, 5), (10, 9)])
def test_zero_gradients_agree_bit_for_bit(shape):
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device")
    from paper_2503_18479_amd import Geometry, Plan, loss_and_grad_many
    t = lambda a: torch.tensor(a, device="cuda:0")
    plans, Cs, Os, Ts = [], [], [], []
    for seed, batch in ((1, 5), (2, 17)):
        wl = W.small_array(*shape, batch=batch, grid=8, n_freq=1, seed=seed)
        plans.append(Plan(Geometry.from_workload(wl.geom), t(wl.pts), wl.bext_z))
        C = t(wl.C)
        C[:, ::3] = float("inf")
        Cs.append(C), Os.append(t(wl.omega)), Ts.append(t(wl.target))
    outs = loss_and_grad_many(plans, Cs, Os, Ts, precision=0)
    for p, C, om, T, out in zip(plans, Cs, Os, Ts, outs):
        loss, grad, st = p.loss_and_grad(C, om, T, precision=0)
        assert int(st.sum()) == 0
        assert torch.equal(grad.view(torch.int64), out[1].view(torch.int64))
        assert torch.equal(loss.view(torch.int64), out[0].view(torch.int64))
        assert not bool(torch.signbit(grad[:, ::3]).any())
