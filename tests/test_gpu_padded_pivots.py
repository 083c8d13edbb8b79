"""Loop counts above 64 that are no multiple of 64, with impedances far above
1 ohm: the identity padding's pivots of 1 are not taken for small ones, so
these systems keep the blocked factorisation, and the results their bound."""
import numpy as np
import pytest

import oracle as O
import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("nx,ny", [(12, 11), (13, 5), (10, 10)])
def test_large_impedances_beside_padding(nx, ny):
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device")
    from paper_2503_18479_amd import Geometry, Plan
    print(f"[padding] {nx * ny} loops", flush=True)
    wl = W.small_array(nx, ny, batch=3, grid=8, n_freq=2, seed=5)
    g, w, C = wl.geom, wl.omega, wl.C * 1e-5  # |Z_kk| of some 10^6 ohm
    t = lambda a: torch.tensor(a, device="cuda:0")
    plan = Plan(Geometry.from_workload(g), t(wl.pts), wl.bext_z)
    M = O.inductance_matrix_fast(g.verts, g.seg_off, g.wire_a)
    Phi = O.flux(g.verts, g.seg_off, wl.bext_z)
    I, st = plan.solve(t(C), t(w))
    Ir = O.currents(M, g.R, Phi, C, w)
    assert int(st.sum()) == 0
    err = np.linalg.norm(I.cpu().numpy() - Ir, axis=2) / np.linalg.norm(Ir, axis=2)
    assert err.max() <= 1e-9
    # the blocked factor is used: the same loops with and without refinement (which
    # only blocked records have) differ in the last bits but not beyond
    plan.set_refinement(True)
    I2, st = plan.solve(t(C), t(w))
    assert int(st.sum()) == 0
    assert float((I2 - I).norm()) <= 1e-11 * float(I.norm())
    assert not torch.equal(I2, I)
