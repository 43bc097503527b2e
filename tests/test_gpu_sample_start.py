"""What a call of the sampler does before its first sweep: W copied in blocks of rows per wave, theta from the spins.

Rows below, at and past the blocks of 1, 2, 5 and 16 waves, one to all of the unit groups in LDS; theta without a sweep
against complex128, N + 1 roundings of 2^-24 of the sum of the terms' magnitudes.  The copy is no longer than one and a
half sweeps of a few chains (the shortest of ten graph replays of 20 calls)."""
import pytest
import torch

import paper_2103_08804_amd as crbm

pytestmark = pytest.mark.gpu


def _state(N, M, C):
    g = torch.Generator("cuda").manual_seed(1000 * N + M)
    c = lambda *s: 0.1 * torch.randn(*s, dtype=torch.complex64, device="cuda", generator=g)
    spins = (2 * torch.randint(0, 2, (C, N), device="cuda", generator=g) - 1).to(torch.int8)
    return crbm.RBM(c(N), c(M), c(N, M)), spins


@pytest.mark.parametrize("C", [1, 300, 1100, 4099])
@pytest.mark.parametrize("N,M", [(2, 1), (7, 64), (8, 65), (9, 150), (17, 200), (33, 300), (40, 400), (64, 512), (127, 449),
                                 (255, 130), (256, 512)])
def test_theta_of_the_start(N, M, C):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    psi, spins = _state(N, M, C)
    plan = crbm.Plan(crbm.CHAIN, N, 1, M, 1)
    theta = torch.full((C, M), float("nan"), dtype=torch.complex64, device="cuda")
    start = spins.clone()
    crbm.sample(plan, psi, spins, 0, crbm.FLIP, 1, 0, theta_out=theta)
    torch.cuda.synchronize()
    plan.close()
    W, b = psi.W.to(torch.complex128), psi.b.to(torch.complex128)
    err = (theta.to(torch.complex128) - (start.to(torch.complex128) @ W + b)).abs()
    assert torch.equal(spins, start)
    assert (err <= (N + 1) * 2.0 ** -24 * (b.abs() + W.abs().sum(0))).all()


@pytest.mark.parametrize("N,M", [(40, 400), (100, 192), (16, 448)])
def test_copy_is_short_for_few_chains(N, M):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    psi, spins = _state(N, M, 4)
    plan, took = crbm.Plan(crbm.CHAIN, N, 1, M, 1), {}
    for sweeps in (0, 8):
        crbm.sample(plan, psi, spins, sweeps, crbm.FLIP, 1, 0)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            for _ in range(20):
                crbm.sample(plan, psi, spins, sweeps, crbm.FLIP, 1, 0)
        best = 1e9
        for _ in range(10):
            t0, t1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            t0.record()
            graph.replay()
            t1.record()
            t1.synchronize()
            best = min(best, t0.elapsed_time(t1) / 20 * 1e3)
        took[sweeps] = best
    plan.close()
    print("us without a sweep", took[0], "per sweep", (took[8] - took[0]) / 8)
    assert took[0] < 1.5 * (took[8] - took[0]) / 8
