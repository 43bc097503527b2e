"""Sign bits of the samples are written with the split of W, in the first launch of a call: rows of whole words, rows of odd
length and rows at an odd address give the same outputs bit for bit, and a plan's second call sees its own samples."""
import numpy as np
import pytest
import torch

import paper_2103_08804_amd as crbm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,M,n", [(4, 1, 1), (12, 70, 65), (33, 5, 300), (64, 130, 257), (256, 40, 129)])
def test_spin_rows(N, M, n):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    g = torch.Generator("cuda").manual_seed(N + M)
    c64 = lambda *s: 0.1 * torch.randn(*s, dtype=torch.complex64, device="cuda", generator=g)
    psi, t = crbm.RBM(c64(N), c64(M), c64(N, M)), c64(1, N + M + N * M)
    betas = torch.ones(1, dtype=torch.complex128, device="cuda")
    raw = torch.zeros(n * N + 1, dtype=torch.int8, device="cuda")
    plan = crbm.Plan(crbm.CHAIN, N, 1, M, n, crbm.PLAN_BASIS, basis_k_max=2)

    def outputs(sig):
        lp, el, T = c64(n), c64(n), c64(n, M)
        mu = torch.zeros(1, 2, dtype=torch.complex128, device="cuda")
        G, H = (torch.zeros(2, 2, dtype=torch.complex128, device="cuda") for _ in range(2))
        crbm.local_estimators(plan, psi, sig, logpsi_out=lp, eloc_out=el, tanh_out=T)
        crbm.chebyshev_moment(plan, psi, t, betas, [(0.3, 0.0)], sig, mu)
        crbm.moment_matrices(plan, psi, t, betas, (0.3, 0.0), sig, G, H)
        return lp, el, T, mu, G, H

    sets = [(2 * torch.randint(0, 2, (n, N), device="cuda", generator=g) - 1).to(torch.int8) for _ in range(2)]
    for sig in sets + sets:
        want = outputs(sig)
        odd = raw[1:].view(n, N)
        odd.copy_(sig)
        assert all(torch.equal(a, b) for a, b in zip(want, outputs(odd)))
        th = sig.to(torch.complex128) @ psi.W.to(torch.complex128) + psi.b.to(torch.complex128)
        assert (want[2] - torch.tanh(th)).abs().max().item() < 1e-4 * (1 + torch.tanh(th).abs().max().item())
    plan.close()
