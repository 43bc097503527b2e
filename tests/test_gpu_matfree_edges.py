"""Matrix-free natural-gradient steps at the edges of the product's tiles, against the factored sums in complex128.

Sites below, at and past the 32, 64, 96 and 128 that a workgroup stages at once, hidden units in the second half of a
tile of 64 and in several tiles, samples that leave partial tiles of 32 and 256, and at N = 130, M = 450 more samples
than one round of the grid takes, so that a workgroup stages W again for a second tile.  S x is formed from the factors,
u = s.x_a + t.(x_b + s x_W), S x = <O^* (u - <u>)>, in complex128.  Tolerances: <O> and F, binary32 operands and chunk
sums, 1e-5 of the largest entry; the solution's residual |(S + eps) x - F| within 32 roundings of 2^-24 of the sums' terms,
tr <O^* O> |x|, and the CG tolerance times |F|."""
import numpy as np
import pytest
import torch

import paper_2103_08804_amd as crbm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,M,n", [(10, 33, 65), (31, 65, 321), (33, 65, 333), (64, 31, 700), (65, 64, 257), (96, 129, 511),
                                   (97, 40, 1000), (128, 63, 289), (130, 70, 515), (256, 100, 1023), (130, 450, 8781)])
@pytest.mark.parametrize("weighted", [False, True])
def test_matfree_step_edges(N, M, n, weighted):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    r = np.random.default_rng(1000 * N + M)
    sig = torch.from_numpy((2 * r.integers(0, 2, size=(n, N)) - 1).astype(np.int8)).cuda()
    T = torch.from_numpy((0.3 * (r.normal(size=(n, M)) + 1j * r.normal(size=(n, M)) + r.normal(size=M)))
                         .astype(np.complex64)).cuda()
    R = torch.from_numpy((1 + 0.3 * r.normal(size=n) + 0.2j * r.normal(size=n)).astype(np.complex64)).cuda()
    w = r.uniform(0.2, 1.0, size=n)
    w = torch.from_numpy(w / w.sum()).cuda() if weighted else None
    plan = crbm.Plan(crbm.CHAIN, N, 1, M, n)
    stats = torch.zeros(8, dtype=torch.float64, device="cuda")
    eps, dg, tol = 1.0, 0.1, 1e-4
    crbm.sr_step(plan, crbm.RBM.empty(N, M), sig, T, R, dg, eps, crbm.CG_MATFREE, crbm.FP32, tol, 200, stats, weights=w)
    F, x, Om = (torch.zeros(plan.P, dtype=torch.complex128, device="cuda") for _ in range(3))
    for which, b in ((crbm.BUF_F, F), (crbm.BUF_DALPHA, x), (crbm.BUF_OMEAN, Om)):
        crbm.copy_plan_buffer(plan, which, b)
    torch.cuda.synchronize()
    assert int(stats[6]) == 0
    s, t, R = sig.to(torch.complex128), T.to(torch.complex128), R.to(torch.complex128)
    w = (w if weighted else torch.full((n,), 1.0 / n, dtype=torch.float64, device="cuda")).to(torch.complex128)

    def contract(c):     # sum_s conj(O_s) c_s
        tc = t.conj().resolve_conj() * c[:, None]
        st = s.T.contiguous()
        return torch.cat([st @ c, tc.sum(0), (st @ tc).reshape(-1)])

    Rm = (w * R).sum()
    gam = np.arccos(min(1.0, abs(Rm.item()) / np.sqrt((w * R.abs() ** 2).sum().real.item())))
    F_ref = dg * gam / np.tan(gam) * contract(w * (R - Rm)) / Rm
    O_ref = contract(w).conj().resolve_conj()
    u = s @ x[:N] + t @ x[N:N + M] + ((s @ x[N + M:].reshape(N, M)) * t).sum(1)
    res = torch.linalg.norm(contract(w * (u - (w * u).sum())) + eps * x - F_ref).item()
    trace = N + (N + 1) * (w.real[:, None] * t.abs() ** 2).sum().item()
    bound = 32 * 2.0 ** -24 * trace * torch.linalg.norm(x).item() + tol * torch.linalg.norm(F_ref).item()
    got = ((Om - O_ref).abs().max() / O_ref.abs().max()).item(), ((F - F_ref).abs().max() / F_ref.abs().max()).item()
    print("N", N, "M", M, "n", n, "means, F:", got, "residual", res, "bound", bound, "iterations", int(stats[5]))
    assert got[0] < 1e-5 and got[1] < 1e-5 and res < bound
    plan.close()
