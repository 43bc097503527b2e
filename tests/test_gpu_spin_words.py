"""Sign bits of the samples below and above the size at which they have a launch of their own (393,216 words past 128
sites): log-derivatives against 64 bits, and two sample sets through one plan."""
import pytest
import torch

import paper_2103_08804_amd as crbm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,M,n", [(129, 3, 78643), (129, 3, 78644), (256, 2, 49153), (128, 2, 98305)])
def test_spin_words(N, M, n):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    g = torch.Generator("cuda").manual_seed(N + n)
    c64 = lambda *s: 0.05 * torch.randn(*s, dtype=torch.complex64, device="cuda", generator=g)
    psi, t = crbm.RBM(c64(N), c64(M), c64(N, M)), c64(1, N + M + N * M)
    betas = torch.ones(1, dtype=torch.complex128, device="cuda")
    raw = torch.zeros(n * N + 1, dtype=torch.int8, device="cuda")
    plan = crbm.Plan(crbm.CHAIN, N, 1, M, n)
    sets = [(2 * torch.randint(0, 2, (n, N), device="cuda", generator=g) - 1).to(torch.int8) for _ in range(2)]

    def moment(sig):
        mu = torch.zeros(1, 2, dtype=torch.complex128, device="cuda")
        crbm.chebyshev_moment(plan, psi, t, betas, [(0.3, 0.0)], sig, mu)
        return mu

    for sig in sets + sets:
        T = c64(n, M)
        mu = moment(sig)
        crbm.local_estimators(plan, psi, sig, tanh_out=T)
        want = torch.tanh(sig.to(torch.complex128) @ psi.W.to(torch.complex128) + psi.b.to(torch.complex128))
        assert (T - want).abs().max().item() < 1e-4 * (1 + want.abs().max().item())
        odd = raw[1:].view(n, N)
        odd.copy_(sig)
        assert torch.equal(moment(odd), mu)
    assert not torch.equal(moment(sets[0]), moment(sets[1]))
    plan.close()
