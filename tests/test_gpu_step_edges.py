"""Natural-gradient steps with the Cholesky solve at the edges of its blocks, against complex128.

P = N + M + N M just below, at and above multiples of the factorisation's 64-column blocks and 16-column panels, and
sample counts that leave the runs of the weighted sums empty, short or uneven.  With weights S is summed in double from
binary32 operands and factored in double as it is: F to 1e-5 and S to 1e-5 of their largest entries (T and R are binary32),
the solution's residual in complex128 within the operands' rounding, 2^-22 of |S + eps I| |x|.  Without weights the
stored binary32 S is factored: the residual on it is below 8 P 2^-53 of |S + eps I| |x| (a backward-stable solve)."""
import numpy as np
import pytest
import torch

import paper_2103_08804_amd as crbm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,M,n", [(2, 4, 3), (3, 3, 16), (2, 5, 17), (7, 7, 64), (4, 12, 65), (10, 5, 129),
                                   (8, 8, 1000), (8, 9, 37), (9, 12, 2048), (11, 15, 511), (10, 23, 4097)])
def test_weighted_step_edges(N, M, n):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    r = np.random.default_rng(100 * N + M + n)
    P = N + M + N * M
    sig = (2 * r.integers(0, 2, size=(n, N)) - 1).astype(np.int8)
    T = (0.5 * (r.normal(size=(n, M)) + 1j * r.normal(size=(n, M)))).astype(np.complex64)
    R = (1 + 0.3 * r.normal(size=n) + 0.2j * r.normal(size=n)).astype(np.complex64)
    w = r.uniform(size=n) ** 4
    w /= w.sum()
    plan = crbm.Plan(crbm.CHAIN, N, 1, M, n, crbm.PLAN_DENSE_S | crbm.PLAN_CHOLESKY)
    dg, eps = 0.1, 1e-2

    def step(weights):
        stats = torch.zeros(8, dtype=torch.float64, device="cuda")
        crbm.sr_step(plan, crbm.RBM.empty(N, M), torch.from_numpy(sig).cuda(), torch.from_numpy(T).cuda(),
                     torch.from_numpy(R).cuda(), dg, eps, crbm.CHOLESKY, crbm.FP32, 1e-10, 1, stats, weights=weights)
        S = torch.zeros(P, P, dtype=torch.complex64, device="cuda")
        F, x, Om = (torch.zeros(P, dtype=torch.complex128, device="cuda") for _ in range(3))
        for which, t in ((crbm.BUF_S, S), (crbm.BUF_F, F), (crbm.BUF_DALPHA, x), (crbm.BUF_OMEAN, Om)):
            crbm.copy_plan_buffer(plan, which, t)
        torch.cuda.synchronize()
        assert int(stats[6]) == 0
        return (t.cpu().numpy().astype(complex) for t in (S, F, x, Om))

    def residual(A, x, F):
        return np.linalg.norm(A @ x - F) / (np.linalg.norm(A) * np.linalg.norm(x))

    S, F, x, Om = step(torch.from_numpy(w).cuda())
    t64, s64, R64 = T.astype(complex), sig.astype(float), R.astype(complex)
    O = np.concatenate([s64, t64, (s64[:, :, None] * t64[:, None, :]).reshape(n, -1)], axis=1)
    m, Rm = w @ O, w @ R64
    gam = np.arccos(min(1.0, abs(Rm) / np.sqrt(w @ np.abs(R64) ** 2)))
    Fr = dg * gam / np.tan(gam) * ((w * (R64 - Rm)) @ O.conj()) / Rm
    C = O - m
    Sr = C.conj().T @ (w[:, None] * C)
    eye = eps * np.eye(P)
    got = (np.abs(Om - m).max(), np.abs(F - Fr).max() / np.abs(Fr).max(), residual(Sr + eye, x, F))
    S, F, x, _ = step(None)
    plan.close()
    Su = (O - O.mean(0)).conj().T @ (O - O.mean(0)) / n
    got += (np.abs(S - Su).max() / np.abs(Su).max(), residual(np.tril(S) + np.tril(S, -1).conj().T + eye, x, F))
    print("P", P, "n", n, "means, F, residual (weighted), S, residual:", got)
    assert got[0] < 1e-6 and got[1] < 1e-5 and got[2] < 2.0 ** -22
    assert got[3] < 1e-5 and got[4] < 8 * P * 2.0 ** -53
