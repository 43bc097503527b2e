"""Dense S from the folded list of tile pairs (hidden blocks hA <= hB, the others mirrored) against complex128.

Shapes at the edges of the tiles: N + 1 extended sites a multiple of 8 (no ragged pairs) or 1, 3, 5 and 6 more
(ragged pairs of 1, 2, 3 live fragments, with and without mixed fragments), M ragged against 16, an odd and an
even count of hidden blocks, and sample counts that leave a partial tile of 128.  Tolerances per entry, on the scale sqrt(S_kk S_k'k') of the centred diagonal: FP32, operands rounded
to 2^-24 and sums of n terms, 4 sqrt(n) 2^-24; BF16, two operands rounded once, 2^-7."""
import numpy as np
import pytest
import torch

import paper_2103_08804_amd as crbm

pytestmark = pytest.mark.gpu

SHAPES = [(23, 53, 1500), (24, 48, 1111), (18, 72, 1290), (20, 67, 1025), (21, 80, 900)]


@pytest.mark.parametrize("N,M,n", SHAPES)
@pytest.mark.parametrize("prec", [crbm.FP32, crbm.BF16])
def test_folded_contraction(N, M, n, prec):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    r = np.random.default_rng(1000 * N + M)
    P = N + M + N * M
    sig = torch.from_numpy((2 * r.integers(0, 2, size=(n, N)) - 1).astype(np.int8)).cuda()
    th = 0.4 * (r.normal(size=(n, M)) + 1j * r.normal(size=(n, M))) + r.normal(size=M)
    T = torch.from_numpy(np.tanh(th).astype(np.complex64)).cuda()
    R = torch.from_numpy((1 + 0.2 * r.normal(size=n) + 0.2j * r.normal(size=n)).astype(np.complex64)).cuda()
    plan = crbm.Plan(crbm.CHAIN, N, 1, M, n, crbm.PLAN_DENSE_S)
    fit = crbm.RBM.empty(N, M)
    stats = torch.zeros(8, dtype=torch.float64, device="cuda")
    crbm.sr_step(plan, fit, sig, T, R, 0.1, 1e-2, crbm.CG_DENSE, prec, 1e-4, 20, stats)
    S = torch.zeros(P, P, dtype=torch.complex64, device="cuda")
    crbm.copy_plan_buffer(plan, crbm.BUF_S, S)
    torch.cuda.synchronize()
    t, s = T.to(torch.complex128), sig.to(torch.complex128)
    O = torch.cat([s, t, (s[:, :, None] * t[:, None, :]).reshape(n, -1)], dim=1)
    O = O - O.mean(0)
    ref = O.mH.contiguous() @ O / n
    d = torch.sqrt(torch.diagonal(ref).real)
    tol = 2.0 ** -7 if prec == crbm.BF16 else 4 * np.sqrt(n) * 2.0 ** -24
    err = ((S.to(torch.complex128) - ref).abs() / (d[:, None] * d[None, :])).max().item()
    print("N", N, "M", M, "n", n, "error", err, "tolerance", tol)
    assert err <= tol
    plan.close()
