"""Impedances so large that the square of a pivot overflows (capacitances far
below any physical one): the currents stay finite and right, also when only
the last pivot of a block is out of range."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("nx,ny,batch", [(8, 8, 2), (16, 8, 3), (12, 12, 2)])
def test_pivots_beyond_the_square_root_of_the_range(nx, ny, batch):
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device")
    from paper_2503_18479_amd import Geometry, Plan
    n = nx * ny
    print(f"[pivot range] {n} loops", flush=True)
    wl = W.small_array(nx, ny, batch=batch, grid=8, n_freq=1, seed=3)
    t = lambda a: torch.tensor(a, device="cuda:0")
    plan = Plan(Geometry.from_workload(wl.geom), t(wl.pts), wl.bext_z)
    w = wl.omega[0]
    Z = np.full((batch, n), 1e152)
    Z[0, -1] = 1e155   # the last pivot alone
    Z[1, 5] = 1e155    # one inside a block
    C = 1.0 / (w * Z)
    I, st = plan.solve(t(C), t(wl.omega))
    I = I.cpu().numpy()[:, 0]
    assert int(st.sum()) == 0
    want = (-1j * w * plan.phi()[None]) / (-1j / (w * C))  # the couplings are 150 orders below
    ok = Z < 1e154
    assert np.all(np.abs(I - want)[ok] <= 1e-9 * np.abs(want)[ok])
    # a reciprocal that underflows may leave no current at all in that loop
    assert np.all(np.abs(I[~ok]) <= (1 + 1e-9) * np.abs(want[~ok]))
