"""Corrected moments and Lanczos at the edges of their in-LDS forms (K < 32, K < 64) and beyond, against numpy.

The basis is K Chebyshev vectors of a random spectrum with a little noise, so that G is well conditioned (below
1e4); both sides work in double, so the tolerance is 1e-9 of mu_0 and of the largest coefficient, as for the other
small dense tests."""
import numpy as np
import pytest
import torch

import paper_2103_08804_amd as crbm
from oracle import spectral

pytestmark = pytest.mark.gpu


def _basis(K, seed=7, D=500, E_c=0.5, W=2.7):
    r = np.random.default_rng(seed + K)
    x = r.uniform(-0.95, 0.95, D)
    V = np.cos(np.arange(K)[:, None] * np.arccos(x)) * np.sqrt(r.uniform(size=D) / D)
    V = V + 1e-3 * (r.normal(size=(K, D)) + 1j * r.normal(size=(K, D)))
    return V.conj() @ V.T, (V.conj() * (E_c + W * x)) @ V.T, E_c, W


def _lanczos(G, H):
    K = G.shape[0]
    Li = np.linalg.inv(np.linalg.cholesky(G))
    Hh = Li @ H @ Li.conj().T
    Q, a, b2 = np.zeros((K, K), complex), np.zeros(K), np.zeros(K)
    Q[0, 0], b2[0] = 1.0, G[0, 0].real
    for j in range(K):
        w = Hh @ Q[j]
        a[j] = (Q[j].conj() @ w).real
        for _ in range(2):
            w = w - Q[:j + 1].T @ (Q[:j + 1].conj() @ w)
        if j + 1 < K:
            b2[j + 1] = np.linalg.norm(w) ** 2
            Q[j + 1] = w / np.sqrt(b2[j + 1])
    return a, b2


@pytest.mark.parametrize("K", [1, 2, 31, 32, 63, 64])
def test_small_dense_edges(K):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    G, H, E_c, W = _basis(K)
    f = dict(dtype=torch.float64, device="cuda")
    plan = crbm.Plan(0, 4, 1, 1, 1)
    Gd, Hd = (torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in (G, H))
    n_out = 2 * K + 3
    mu, info = torch.zeros(n_out, **f), torch.zeros(3, **f)
    crbm.corrected_moments(plan, Gd, Hd, E_c, W, mu, info)
    a, b2, li = torch.zeros(K, **f), torch.zeros(K, **f), torch.zeros(2, **f)
    crbm.lanczos(plan, Gd, Hd, a, b2, li)
    torch.cuda.synchronize()
    assert int(info[0]) == 0 and int(li[0]) == 0 and int(li[1]) == K
    ref = spectral.corrected_moments(G, H, E_c, W, n_out)
    ra, rb = _lanczos(G, H)
    err = (np.abs(mu.cpu().numpy() - ref).max() / abs(ref[0]), np.abs(a.cpu().numpy() - ra).max() / np.abs(ra).max(),
           np.abs(b2.cpu().numpy() - rb).max() / np.abs(rb).max())
    print("K", K, "cond G", np.linalg.cond(G), "errors", err)
    assert max(err) < 1e-9


@pytest.mark.parametrize("n_mom,n_w", [(1, 3), (2, 64), (512, 65), (513, 130), (1030, 7)])
def test_kpm_chunks(n_mom, n_w):
    """The coefficients are formed 512 moments at a time and a block takes 64 frequencies."""
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    r = np.random.default_rng(n_mom)
    mu = r.normal(size=n_mom) / (1 + np.arange(n_mom))
    om = np.linspace(-0.5, 6.0, n_w)
    f = dict(dtype=torch.float64, device="cuda")
    A = torch.zeros(n_w, **f)
    crbm.spectrum_kpm(torch.from_numpy(mu).cuda(), -2.0, 0.5, 2.7, torch.from_numpy(om).cuda(), A)
    torch.cuda.synchronize()
    ref = spectral.kpm_spectrum(mu, -2.0, 0.5, 2.7, om)
    assert np.max(np.abs(A.cpu().numpy() - ref)) < 1e-9 * max(np.max(np.abs(ref)), 1e-30)
