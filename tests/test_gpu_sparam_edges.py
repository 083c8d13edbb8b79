"""The S-parameter solver and one-pass contraction at their edges, against the
oracle: port counts around 16, 32 and 48, where the contraction's extent and
the solver's two column halves change; points around its tiles of 16; a batch
beyond the factor record's 131,072 systems (factored in slabs); batches that
shrink below a reserved one; and zero pivots that need row exchanges."""
import numpy as np
import pytest

from oracle import sparam_oracle as SO
from test_gpu_sparam import TOL, _general, _nrel, _plan

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device")
    return torch.device("cuda:0")


def _check(dev, pl, S0, fields, scc, ix, iy, vals, exc, T, n0, comp, prec=0, mode=0):
    t = lambda a: torch.tensor(a, device=dev)
    loss, g, st = pl.loss_and_grad(t(vals), t(T), comp, mode, prec)
    assert int(st.abs().sum()) == 0
    SC = SO.assemble_network(scc, vals, ix, iy)
    Lr = SO.loss(SO.combine(S0, fields, SC, n0, exc)[1], T, comp, mode)
    gr = SO.grad_adjoint(S0, fields, SC, n0, exc, ix, iy, T, comp, mode)
    assert np.max(np.abs(loss.cpu().numpy() - Lr) / Lr) < TOL[prec]
    assert _nrel(g.cpu().numpy(), gr) < TOL[prec]


@pytest.mark.parametrize("n0,P", [(2, 1), (15, 15), (16, 16), (17, 17), (31, 33), (32, 64), (33, 100),
                                  (48, 47), (49, 1000), (63, 31), (64, 16)])
def test_ports_and_points(dev, n0, P):
    print(f"[sp edges] {n0} ports, {P} points", flush=True)
    S0, fields, scc, ix, iy, vals, exc, T = _general(n0, 67, 2, n0, 2, P, 2)
    pl = _plan(dev, S0, fields, scc, ix, iy, exc)
    for prec in (0, 1):
        _check(dev, pl, S0, fields, scc, ix, iy, vals, exc, T, n0, 1, prec, n0 % 2)
    pl.reserve(300)
    for B in (1, 5, 64):
        _check(dev, pl, S0, fields, scc, ix, iy, vals[:B], exc, T, n0, 0)


def test_zero_diagonal_needs_pivoting(dev):
    """A matrix whose leading pivots vanish: constant entries cancel the unit
    diagonal of I - S_C11 S0 in the first rows."""
    n0, F, P = 34, 1, 20
    S0, fields, scc, ix, iy, vals, exc, T = _general(91, 3, F, n0, 1, P, 1)
    # S_C11,const S0 = I + a cyclic shift in rows 0..9, so that row k of A starts
    # with a zero on the diagonal; the variable entries stay off those rows
    target = np.zeros((n0, n0), complex)
    for k in range(10):
        target[k, k] = 1.0
        target[k, (k + 1) % 10] = -0.7 - 0.2j
    scc[0, :10, :n0] = np.linalg.solve(S0[0].T, target[:10].T).T
    keep = ix >= 10
    ix, iy, vals = ix[keep], iy[keep], np.ascontiguousarray(vals[:, :, keep])
    pl = _plan(dev, S0, fields, scc, ix, iy, exc)
    _check(dev, pl, S0, fields, scc, ix, iy, vals, exc, T, n0, 0)


def test_more_systems_than_the_record_holds(dev):
    n0, B = 3, 131072 + 700
    S0, fields, scc, ix, iy, _, exc, T = _general(5, 1, 1, n0, 1, 3, 1)
    rng = np.random.default_rng(6)
    vals = 0.6 * np.exp(1j * rng.uniform(0, 2 * np.pi, (B, 1, len(ix))))
    pl = _plan(dev, S0, fields, scc, ix, iy, exc, prec=("fp64",))
    loss, g, st = pl.loss_and_grad(torch.tensor(vals, device=dev), torch.tensor(T, device=dev), 0, 0, 0)
    assert int(st.abs().sum()) == 0
    pick = [0, 1, 70000, 131071, 131072, B - 1]
    SC = SO.assemble_network(scc, vals[pick], ix, iy)
    Lr = SO.loss(SO.combine(S0, fields, SC, n0, exc)[1], T, 0, 0)
    gr = SO.grad_adjoint(S0, fields, SC, n0, exc, ix, iy, T, 0, 0)
    assert np.max(np.abs(loss.cpu().numpy()[pick] - Lr) / Lr) < 1e-9
    assert _nrel(g.cpu().numpy()[pick], gr) < 1e-9
