"""Fidelity gradient where the grouping of its contraction changes: sample chunks of 128 and 256, one to four blocks of
32 sites per wave, and sample counts at the edges of both, against complex128.

FP32 sums of at most 256 terms: 4 sqrt(256) 2^-24 of the sum of the terms' magnitudes, per entry.  The gradient without
a plan groups alike, so it is the same bit for bit.  Few samples leave most of the device idle, so the time of a call is
one workgroup's walk through its chunk: on four site blocks it stays within 1.4 times that on one."""
import numpy as np
import pytest
import torch

import paper_2103_08804_amd as crbm

pytestmark = pytest.mark.gpu


def _inputs(N, M, n):
    g = torch.Generator("cuda").manual_seed(1000 * N + M + n)
    sig = (2 * torch.randint(0, 2, (n, N), device="cuda", generator=g) - 1).to(torch.int8)
    T = 0.4 * torch.randn(n, M, dtype=torch.complex64, device="cuda", generator=g)
    return sig, T, 1 + 0.3 * torch.randn(n, dtype=torch.complex64, device="cuda", generator=g)


@pytest.mark.parametrize("N,M,n", [(5, 3, 1), (31, 31, 127), (32, 31, 128), (40, 5, 129), (33, 130, 257), (64, 72, 385),
                                   (100, 128, 3072), (100, 400, 3073), (100, 400, 8193), (200, 200, 2305), (256, 512, 1024),
                                   (256, 512, 4100), (31, 31, 49152), (31, 31, 49153)])
def test_gradient_groups(N, M, n):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    sig, T, R = _inputs(N, M, n)
    P = N + M + N * M
    plan = crbm.Plan(crbm.CHAIN, N, 1, M, n)
    g, g2 = (torch.full((P,), float("nan"), dtype=torch.complex128, device="cuda") for _ in range(2))
    crbm.fidelity_grad(plan, crbm.RBM.empty(N, M), sig, T, R, g)
    crbm.fidelity_grad_noalloc(N, M, sig, T, R, g2)
    torch.cuda.synchronize()
    plan.close()
    s, t, R = sig.to(torch.complex128), T.to(torch.complex128), R.to(torch.complex128)
    c = 2 * (1 - R) * R.conj() / n
    st = s.T.contiguous()
    cat = lambda a, tc: torch.cat([st @ a, tc.sum(0), (st @ tc).reshape(-1)])
    ref = cat(c, t.conj() * c[:, None])
    tc = (t.abs() * c.abs()[:, None]).sum(0)
    scale = torch.cat([c.abs().sum().expand(N), tc, tc.repeat(N)])
    err = ((g - ref).abs() / scale).max().item()
    print("N", N, "M", M, "n", n, "error", err)
    assert torch.equal(g, g2)
    assert err <= 4 * np.sqrt(256) * 2.0 ** -24


def test_few_samples_do_not_wait_for_site_blocks():
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")

    def per_call(N, M, n, calls=20):
        sig, T, R = _inputs(N, M, n)
        plan, fit = crbm.Plan(crbm.CHAIN, N, 1, M, n), crbm.RBM.empty(N, M)
        out = torch.zeros(N + M + N * M, dtype=torch.complex128, device="cuda")
        crbm.fidelity_grad(plan, fit, sig, T, R, out)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            for _ in range(calls):
                crbm.fidelity_grad(plan, fit, sig, T, R, out)
        best = 1e9
        for _ in range(10):
            t0, t1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            t0.record()
            graph.replay()
            t1.record()
            t1.synchronize()
            best = min(best, t0.elapsed_time(t1) / calls * 1e3)
        plan.close()
        return best

    one, four = per_call(20, 16, 300), per_call(100, 16, 300)
    print("us per gradient on one and four site blocks:", one, four)
    assert four < 1.4 * one
