"""The factor record of a solve ends when the refinement mode changes: the FP64
and the FP32 factor are kept in different types and places, so a replay in
the other mode is refused on the host, and a new solve makes a new record."""
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("nx,ny", [(10, 10), (4, 4)])
@pytest.mark.parametrize("first", [False, True])
def test_mode_change_ends_the_record(nx, ny, first):
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device")
    from paper_2503_18479_amd import CosimError, Geometry, Plan
    print(f"[record] {nx * ny} loops, refinement {first} -> {not first}", flush=True)
    dev = torch.device("cuda:0")
    wl = W.small_array(nx, ny, batch=3, grid=9, n_freq=2, seed=nx)
    t = lambda a: torch.tensor(a, device=dev)
    plan = Plan(Geometry.from_workload(wl.geom), t(wl.pts), wl.bext_z)
    C, om = t(wl.C), t(wl.omega)
    gB = torch.ones((3, 2, plan.P), dtype=torch.complex128, device=dev)
    plan.set_refinement(first)
    I, _ = plan.solve(C, om)
    want, _ = plan.field_backward(C, om, I, gB, reuse=True)
    plan.set_refinement(not first)
    with pytest.raises(CosimError) as e:
        plan.field_backward(C, om, I, gB, reuse=True)
    assert e.value.code == -1  # COSIM_EINVAL, before anything is enqueued
    I, _ = plan.solve(C, om)
    got, _ = plan.field_backward(C, om, I, gB, reuse=True)
    # both modes meet 1e-11 of FP64 (refinement to 1e-12, then one product)
    assert float((got - want).norm()) <= 1e-10 * float(want.norm())
