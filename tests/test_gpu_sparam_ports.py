"""The S-parameter solver where the number of columns that its steps carry
changes (multiples of 8 ports, in either half of 32 columns), forward and with
gradients, against the oracle, one system of the batch being NaN."""
import numpy as np
import pytest

from oracle import sparam_oracle as SO
from test_gpu_sparam import TOL, _general, _nrel, _plan

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n0", [1, 7, 8, 9, 24, 25, 40, 41, 47, 56, 57])
def test_columns_of_the_solver(n0):
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device")
    dev = torch.device("cuda:0")
    print(f"[sp ports] {n0} ports", flush=True)
    B, F = 6, 2
    S0, fields, scc, ix, iy, vals, exc, T = _general(200 + n0, B, F, n0, 2, 9, 1)
    t = lambda a: torch.tensor(a, device=dev)
    pl = _plan(dev, S0, fields, scc, ix, iy, exc)
    SC = SO.assemble_network(scc, vals, ix, iy)
    xr, Br = SO.combine(S0, fields, SC, n0, exc)
    Lr = SO.loss(Br, T, 0, 0)
    gr = SO.grad_adjoint(S0, fields, SC, n0, exc, ix, iy, T, 0, 0)
    v = vals.copy()
    v[3, 1, 0] = np.nan  # system (3, 1) alone
    rest = [0, 1, 2, 4, 5]
    x, Bc, st = pl.field(t(v))
    x, Bc = x.cpu().numpy(), Bc.cpu().numpy()
    assert int(st[3, 1]) == 4 and int(st.sum()) == 4
    assert _nrel(x[rest], xr[rest]) < TOL[0] and _nrel(x[3, 0], xr[3, 0]) < TOL[0]
    assert _nrel(Bc[rest], Br[rest]) < TOL[0] and np.isnan(x[3, 1]).any()
    for prec in (0, 1):
        loss, g, st = pl.loss_and_grad(t(v), t(T), 0, 0, prec)
        assert int(st.sum()) == 4 and bool(torch.isnan(loss[3]))
        assert np.max(np.abs(loss.cpu().numpy()[rest] - Lr[rest]) / Lr[rest]) < TOL[prec]
        assert _nrel(g.cpu().numpy()[rest], gr[rest]) < TOL[prec]
