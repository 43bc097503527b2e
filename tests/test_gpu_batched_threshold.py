"""The acceptance threshold of the batched moments at its last bit, on every launch shape.

With W = b = 0 of psi_gs a move changes no log cosh, so a flip of site i (an exchange of i and j) from spin s_i is
accepted when ln(u)/2 + s_i d2 < 0, d2 = 2 Re a_i (2 Re (a_i - a_j)).  Re a puts |d2| one unit in the last place below,
at and above the rounded |ln(u)/2| of chosen first proposals: at N <= 64 the product (ln 2 / 2) log2 u and the sum round
once together, so the decision is that of the exact product; at N > 64 the product rounds first and a draw on the rounded
value is rejected.  log2 u is the device's; the rest is exact in double (24 x 24 bit products)."""
import numpy as np
import pytest
import torch

import paper_2103_08804_amd as crbm

pytestmark = pytest.mark.gpu

HALF_LN2 = float(np.float32(0.34657359027997264))
SEED = 77


def _first_draws(orc, N, total):
    """Sites i, j and the uniform of proposal 0 of every chain (counter (chain, 0, 0), tag 0)."""
    x = np.array([orc.philox([g, 0, 0, 0], [SEED, 0]) for g in range(total)], dtype=np.uint64)
    return (x[:, 0] * N >> 32).astype(int), (x[:, 1] * N >> 32).astype(int), ((x[:, 2] >> 8) / 2.0 ** 24).astype(np.float32)


@pytest.mark.parametrize("N,M,proposal", [(16, 16, 1), (64, 70, 0), (64, 128, 1), (64, 300, 1), (66, 70, 0),
                                          (66, 128, 1), (100, 200, 1)])
def test_threshold_last_bit(orc, N, M, proposal):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    total, P = 1024, N + M + N * M
    i, j, u = _first_draws(orc, N, total)
    lu = HALF_LN2 * torch.log2(torch.from_numpy(u).cuda()).cpu().numpy().astype(np.float64)   # exact product
    plan = crbm.Plan(crbm.CHAIN, N, 1, M, total)
    spins = torch.zeros(total, N, dtype=torch.int8, device="cuda")
    crbm.init_chains(plan, spins, SEED, True)
    s0 = spins.cpu().numpy()
    r = np.random.default_rng(N + M)
    t = torch.from_numpy((0.05 * (r.normal(size=(1, P)) + 1j * r.normal(size=(1, P)))).astype(np.complex64)).cuda()
    beta = torch.ones(1, dtype=torch.complex128, device="cuda")
    q = torch.zeros(1, 2, dtype=torch.float64, device="cuda")
    off = torch.tensor([0, total], dtype=torch.int64, device="cuda")
    shapes = [(w, b, ln) for ln in (64, 32, 16) if ln == 64 or (ln == 32 and M <= 256) or M <= 128
              for w, b in ((1, 3), (8, 512))]
    zero = lambda *s: torch.zeros(*s, dtype=torch.complex64, device="cuda")
    live = (u > 2.0 ** -20) & (np.ones(total, bool) if proposal == 0 else s0[np.arange(total), i] != s0[np.arange(total), j])
    chains, told_apart = np.flatnonzero(live), 0
    while chains.size and told_apart < 12:
        # chains whose first proposals touch sites of their own
        used, pick, rest = set(), [], []
        for g in chains:
            sites = {i[g]} if proposal == 0 else {i[g], j[g]}
            (rest if used & sites else pick).append(g)
            if pick and pick[-1] == g:
                used |= sites
        chains, pick = np.array(rest, dtype=int), np.array(pick)
        for ulps in (-1, 0, 1):
            near = np.abs(lu[pick].astype(np.float32))
            d2 = (near + ulps * np.spacing(near)).astype(np.float32)
            a = np.zeros(N, np.complex64)
            a[i[pick]] = 0.5 * s0[pick, i[pick]] * d2
            fused = lu[pick] + d2.astype(np.float64) < 0
            rounded = lu[pick].astype(np.float32) + d2 < 0
            told_apart += int((fused != rounded).sum())
            gs = crbm.RBM(torch.from_numpy(a).cuda(), zero(M), zero(N, M))
            first = None
            for w, b, ln in shapes:
                crbm.batched_set_shape(plan, w, b, ln)
                mu = torch.zeros(1, 2, dtype=torch.complex128, device="cuda")
                tr = torch.zeros(total, (N + 31) // 32, dtype=torch.int32, device="cuda")
                crbm.batched_moments(plan, gs, t, beta, q, off, 0, 1, proposal, SEED, mu, total_chains=total, trace=tr)
                bits = (tr[:, 0] & 1).bool().cpu().numpy()[pick]
                assert np.array_equal(bits, fused if N <= 64 else rounded), (w, b, ln, ulps)
                first = (mu, tr) if first is None else first
                assert torch.equal(mu, first[0]) and torch.equal(tr, first[1]), (w, b, ln, ulps)
    print("N", N, "M", M, "decisions that tell the two roundings apart:", told_apart)
    assert told_apart >= 8
    plan.close()
