"""Sample splits of the dense S contraction pay for their slices: in BF16 a contraction of few samples is not split so far
that adding the slices takes as long as forming them (the time of the plan's kernel groups, the smallest of five steps)."""
import pytest
import torch

import paper_2103_08804_amd as crbm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,Lx,Ly,M,n", [(1, 10, 10, 72, 1000), (1, 10, 10, 40, 4000), (1, 8, 8, 72, 4000)])
def test_slices_cost_less_than_the_contraction(kind, Lx, Ly, M, n):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    N = Lx * Ly
    g = torch.Generator("cuda").manual_seed(N + M)
    sig = (2 * torch.randint(0, 2, (n, N), device="cuda", generator=g) - 1).to(torch.int8)
    T = 0.3 * torch.randn(n, M, dtype=torch.complex64, device="cuda", generator=g)
    R = 1 + 0.1 * torch.randn(n, dtype=torch.complex64, device="cuda", generator=g)
    stats = torch.zeros(8, dtype=torch.float64, device="cuda")
    plan, fit = crbm.Plan(kind, Lx, Ly, M, n, crbm.PLAN_DENSE_S), crbm.RBM.empty(N, M)
    sums, products = [], []
    for _ in range(6):
        plan.profile(True)
        crbm.sr_step(plan, fit, sig, T, R, 0.1, 1e-2, crbm.CG_DENSE, crbm.BF16, 1e-3, 1, stats)
        torch.cuda.synchronize()
        t = plan.profile_read()
        plan.profile(False)
        sums.append(t["sborder"][1])      # the border sums and the slices
        products.append(t["sbuild"][1])
    plan.close()
    print("N", N, "M", M, "n", n, "slices and border", min(sums[1:]), "ms, contraction", min(products[1:]), "ms")
    assert min(sums[1:]) < 0.7 * min(products[1:])
