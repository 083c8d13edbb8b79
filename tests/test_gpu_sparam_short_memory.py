"""An S-parameter batch whose factor record does not fit beside what the program
holds: the record is made smaller, the results stay the same bits."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

GB = 1 << 30


def test_record_in_slabs_when_memory_is_short():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device")
    from paper_2503_18479_amd import SParamPlan, trim
    dev = torch.device("cuda:0")
    n0, F, P, B = 64, 2, 16, 50000  # a record of 6.5 GB
    gen = torch.Generator(device=dev).manual_seed(1)
    rnd = lambda *s: torch.randn(*s, dtype=torch.complex128, device=dev, generator=gen)
    S0, fields = 0.05 * rnd(F, n0, n0), rnd(F, P, 1, n0)
    ix = np.arange(n0, dtype=np.int32)
    values = 0.6 * torch.exp(6.28j * torch.rand(B, F, n0, dtype=torch.float64, device=dev, generator=gen))
    T = torch.rand(P, dtype=torch.float64, device=dev, generator=gen)
    sc = 0.05 * rnd(F, n0 + 1, n0 + 1)
    make = lambda: SParamPlan(S0, fields, ix, ix, np.ones(1), sc_const=sc, precisions=["fp64"])
    plan = make()
    want = plan.loss_and_grad(values, T)
    del plan
    trim()
    torch.cuda.synchronize()
    held = []
    try:
        while torch.cuda.mem_get_info()[0] > 5 * GB // 2:
            free = torch.cuda.mem_get_info()[0]
            held.append(torch.empty(min(32 * GB, free - 9 * GB // 4), dtype=torch.uint8, device=dev))
        print(f"[short memory] {torch.cuda.mem_get_info()[0] / GB:.2f} GB left", flush=True)
        plan = make()
        got = plan.loss_and_grad(values, T)
        assert all(torch.equal(a, b) for a, b in zip(got, want))
    finally:
        del held
        torch.cuda.empty_cache()
