"""The contraction over samples sum_s sigma~_i(s) c(s) conj(t~_j(s)) through the fidelity gradient, against complex128.

Shapes at the edges of its tiles: N + 1 extended sites in 1 to 9 blocks of 32 (equal groups of at most four, the last
group partly empty), M + 1 extended units in 1 to 17 blocks of 32 (one to four waves), sample counts at 16-sample steps,
64-sample words, coefficient tiles and 256-sample chunks, sample rows at odd addresses.  Binary32 sums of n terms per
chunk of c = max(256, n / 256) samples, each term rounded three times: error at most (c + 3) 2^-24 sum_s |c| |t~|; and
an infinite ratio gives no finite entry in its columns."""
import numpy as np
import pytest
import torch

import paper_2103_08804_amd as crbm

pytestmark = pytest.mark.gpu


def _run(N, M, n, shift, R, T, sig):
    raw = torch.zeros(n * N + shift, dtype=torch.int8, device="cuda")
    s = raw[shift:].view(n, N)
    s.copy_(torch.from_numpy(sig))
    plan = crbm.Plan(crbm.CHAIN, N, 1, M, n)
    grad = torch.zeros(N + M + N * M, dtype=torch.complex128, device="cuda")
    crbm.fidelity_grad(plan, crbm.RBM.empty(N, M), s, torch.from_numpy(T).cuda(), torch.from_numpy(R).cuda(), grad)
    torch.cuda.synchronize()
    plan.close()
    return grad.cpu().numpy()


@pytest.mark.parametrize("N,M,n,shift", [
    (2, 1, 1, 0), (31, 31, 17, 1), (32, 32, 64, 0), (33, 63, 65, 3), (64, 96, 255, 0), (95, 127, 256, 1),
    (96, 128, 257, 0), (128, 160, 300, 2), (150, 40, 777, 0), (160, 255, 511, 0), (200, 300, 1000, 1),
    (256, 512, 513, 0), (12, 20, 70001, 0)])
def test_gradient_edges(N, M, n, shift):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    r = np.random.default_rng(N * M + n)
    sig = (2 * r.integers(0, 2, size=(n, N)) - 1).astype(np.int8)
    T = (r.normal(size=(n, M)) + 1j * r.normal(size=(n, M))).astype(np.complex64)
    R = (1 + 0.3 * (r.normal(size=n) + 1j * r.normal(size=n))).astype(np.complex64)
    got = _run(N, M, n, shift, R, T, sig)
    c = 2 * (1 - R.astype(complex)) * R.conj().astype(complex) / n
    t1 = np.concatenate([T.astype(complex), np.ones((n, 1))], axis=1).conj()
    s1 = np.concatenate([sig, np.ones((n, 1), np.int8)], axis=1).astype(float)
    ref = s1.T @ (c[:, None] * t1)                      # [N + 1][M + 1]
    scale = (np.abs(c)[:, None] * np.abs(t1)).sum(0)    # per column
    tol = (max(256, n / 256) + 3) * 2.0 ** -24 * scale
    err = np.abs(np.concatenate([got[:N] - ref[:N, M], got[N:N + M] - ref[N, :M], (got[N + M:].reshape(N, M) - ref[:N, :M]).ravel()]))
    lim = np.concatenate([np.full(N, tol[M]), tol[:M], np.broadcast_to(tol[:M], (N, M)).ravel()])
    print("N", N, "M", M, "n", n, "largest error over its limit", (err / lim).max())
    assert np.all(err <= lim)


def test_infinite_unit():
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    N, M, n = 6, 40, 100
    r = np.random.default_rng(1)
    sig = (2 * r.integers(0, 2, size=(n, N)) - 1).astype(np.int8)
    T = (r.normal(size=(n, M)) + 0j).astype(np.complex64)
    T[50, 7] = np.inf
    got = _run(N, M, n, 0, np.full(n, 0.5, np.complex64), T, sig)
    W = got[N + M:].reshape(N, M)
    assert not np.isfinite(W[:, 7]).any() and np.isfinite(np.delete(W, 7, axis=1)).all()
    assert np.isfinite(got[:N]).all() and not np.isfinite(got[N + 7])
