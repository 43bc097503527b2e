"""A plan is ready when its creation returns: its first call, on a stream that does not wait for the null stream, gives what
later calls give, estimators (the split of W) and matrix-free steps (its padding) alike."""
import pytest
import torch

import paper_2103_08804_amd as crbm

pytestmark = pytest.mark.gpu


def test_first_call_on_another_stream():
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    N, M, n = 130, 450, 300
    g = torch.Generator("cuda").manual_seed(3)
    c = lambda *s: 0.05 * torch.randn(*s, dtype=torch.complex64, device="cuda", generator=g)
    psi, R = crbm.RBM(c(N), c(M), c(N, M)), 1 + c(n)
    sig = (2 * torch.randint(0, 2, (n, N), device="cuda", generator=g) - 1).to(torch.int8)
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    want = None
    for _ in range(10):
        plan = crbm.Plan(crbm.CHAIN, N, 1, M, n)
        with torch.cuda.stream(side):
            T, fit = torch.zeros(n, M, dtype=torch.complex64, device="cuda"), crbm.RBM.empty(N, M)
            stats = torch.zeros(8, dtype=torch.float64, device="cuda")
            crbm.local_estimators(plan, psi, sig, tanh_out=T)
            crbm.sr_step(plan, fit, sig, T, R, 0.1, 1e-2, crbm.CG_MATFREE, crbm.FP32, 1e-6, 20, stats)
        side.synchronize()
        plan.close()
        got = (T, stats, fit.W)
        want = got if want is None else want
        assert all(torch.equal(a, b) for a, b in zip(got, want))
    assert torch.isfinite(want[1]).all()
