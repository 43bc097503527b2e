"""Chebyshev moments at the edges of the fused product's tiles, against complex128.

Sites in the second, third and last of the pieces of W that a workgroup stages and in every word of sign bits, hidden
units in partial and several tiles of 64, odd sample counts, and at N = 130, M = 450 more samples than one round of the
grid takes.  A moment is a mean of f^* B with B = beta t / psi_gs: every log psi is a binary32 sum of terms of total
size L with at most 8 roundings in a row (2^-24 each), two of them in a ratio, so the error stays below
16 2^-24 (L_t + L_gs) of the mean of |f| |B|."""
import numpy as np
import pytest
import torch

import paper_2103_08804_amd as crbm
from gpu_util import EPS32

pytestmark = pytest.mark.gpu


def _log_psi(v, s, N, M):
    """log psi (up to the M log 2 of log 2 cosh) and the size of its terms, in complex128."""
    a, b, W = v[:N], v[N:N + M], v[N + M:].reshape(N, M)
    th = s @ W + b
    flip = torch.where(th.real >= 0, 1.0, -1.0)
    z = th * flip
    lc = z + torch.log((1 + torch.exp(-2 * z)) / 2)
    asig = s @ a
    return lc.sum(1) + asig, (th.abs().sum(1) + asig.abs()).max().item()


@pytest.mark.parametrize("N,M,n", [(3, 5, 7), (33, 31, 77), (40, 80, 1001), (65, 65, 259), (90, 64, 513), (97, 130, 301),
                                   (128, 33, 255), (130, 70, 1031), (225, 20, 129), (256, 100, 767), (130, 450, 8781)])
def test_moment_edges(N, M, n):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    r = np.random.default_rng(1000 * N + M + n)
    P, n_max = N + M + N * M, 2
    draw = lambda k, sd: torch.from_numpy((sd * (r.normal(size=(k, P)) + 0.3j * r.normal(size=(k, P)))).astype(np.complex64))
    gs, t = draw(1, 0.03)[0].cuda(), draw(n_max, 0.03).cuda()
    sig = torch.from_numpy((2 * r.integers(0, 2, size=(n, N)) - 1).astype(np.int8)).cuda()
    w = r.uniform(0.2, 1.0, size=n)
    w = torch.from_numpy(w / w.sum()).cuda()
    betas = torch.from_numpy(r.normal(size=n_max) + 1j * r.normal(size=n_max)).cuda()
    qs = [(0.0, 0.0), (2 * np.pi / N, 0.0), (np.pi, 0.0)]
    mu = torch.zeros(len(qs), n_max + 1, dtype=torch.complex128, device="cuda")
    plan = crbm.Plan(crbm.CHAIN, N, 1, M, n)
    rbm = crbm.RBM(gs[:N].contiguous(), gs[N:N + M].contiguous(), gs[N + M:].reshape(N, M).contiguous())
    crbm.chebyshev_moment(plan, rbm, t, betas, qs, sig, mu, weights=w)
    torch.cuda.synchronize()
    plan.close()
    s = sig.to(torch.complex128)
    x = torch.arange(N, device="cuda", dtype=torch.float64)
    f = [s @ torch.exp(-1j * q[0] * x) / (2 * np.sqrt(N)) for q in qs]
    lg, Lg = _log_psi(gs.to(torch.complex128), s, N, M)
    worst = 0.0
    for iq in range(len(qs)):
        ref = (w * f[iq].abs() ** 2).sum()
        assert abs(mu[iq, 0] - ref).item() <= 1e-12 * ref.real.item()
    for k in range(n_max):
        lt, Lt = _log_psi(t[k].to(torch.complex128), s, N, M)
        B = betas[k] * torch.exp(lt - lg)
        for iq in range(len(qs)):
            ref, scale = (w * f[iq].conj() * B).sum(), (w * f[iq].abs() * B.abs()).sum().item()
            worst = max(worst, abs(mu[iq, k + 1] - ref).item() / (16 * EPS32 * (Lt + Lg) * scale))
    print("N", N, "M", M, "n", n, "error over bound", worst)
    assert worst <= 1.0
