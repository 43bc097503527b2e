"""Metropolis sweeps at the edges of their work split, replayed by the oracle decision for decision.

Proposals are drawn 64 at a time, so sweeps shorter and longer than that end inside a batch and the last batch is
partial; M takes 1 to 8 unit groups of 64, of which one, two, three or all sit in LDS; 1 to 16 chains share a
workgroup, the last of which may be partly filled; rows of N sites start at odd addresses or not, and are stored four
sites at a time where they can be."""
import numpy as np
import pytest
import synth
import torch

import paper_2103_08804_amd as crbm
from gpu_util import np_of, rel_err, to_device_rbm, to_oracle_rbm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,M,C,sweeps,proposal,std,shift", [
    (3, 64, 5, 30, 0, 0.3, 0), (62, 65, 300, 3, 1, 0.1, 1), (64, 129, 257, 2, 1, 0.1, 0), (66, 200, 70, 2, 0, 0.05, 2),
    (40, 300, 513, 2, 1, 0.05, 0), (160, 321, 20, 1, 1, 0.03, 0), (110, 450, 33, 2, 1, 0.03, 3),
    (256, 512, 9, 1, 0, 0.02, 0), (24, 512, 18, 3, 1, 0.05, 1), (10, 70, 4100, 2, 1, 0.2, 0)])
def test_sweep_edges(orc, N, M, C, sweeps, proposal, std, shift):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    psi_d = to_device_rbm(orc.RBM(*synth.random_rbm_arrays(N + M, N, M, std, std_im=0.02)))
    psi = to_oracle_rbm(orc, psi_d)
    plan = crbm.Plan(crbm.CHAIN, N, 1, M, 1)
    raw = [torch.zeros(k * C * N + shift, dtype=torch.int8, device="cuda")[shift:] for k in (1, sweeps)]
    spins, samples = raw[0].view(C, N), raw[1].view(sweeps, C, N)
    crbm.init_chains(plan, spins, 2000 + N, proposal == 1 and N % 2 == 0)
    s_ref = np_of(spins).copy()
    nacc = torch.zeros(C, dtype=torch.int32, device="cuda")
    trace = torch.full((C, (sweeps * N + 31) // 32), -1, dtype=torch.int32, device="cuda")
    theta = torch.zeros(C, M, dtype=torch.complex64, device="cuda")
    crbm.sample(plan, psi_d, spins, sweeps, proposal, 7 + N, 99, theta_out=theta, samples_out=samples, n_accept=nacc,
                trace=trace)
    torch.cuda.synchronize()
    smp_ref, nacc_ref, amb, mis = orc.metropolis(psi, s_ref, sweeps, proposal, 7 + N, 99,
                                                 trace=np_of(trace).view(np.uint32))
    assert mis == 0 and amb <= max(3, 1e-3 * sweeps * N * C)
    assert np.array_equal(np_of(samples), smp_ref)
    assert np.array_equal(np_of(spins), s_ref)
    assert np.array_equal(np_of(nacc).view(np.uint32), nacc_ref)
    assert rel_err(np_of(theta), psi.b[None, :] + s_ref.astype(np.float64) @ psi.W) < 1e-5
    plan.close()


def test_sweep_in_a_graph(orc):
    """A sweep whose copy of W takes more than 64 KB of LDS, captured on its first call and replayed."""
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    N, M, C = 100, 400, 64
    psi = to_device_rbm(orc.RBM(*synth.random_rbm_arrays(3, N, M, 0.03, std_im=0.02)))
    plan = crbm.Plan(crbm.CHAIN, N, 1, M, 1)
    start = torch.zeros(C, N, dtype=torch.int8, device="cuda")
    crbm.init_chains(plan, start, 5, True)
    spins, out = start.clone(), torch.zeros(2, C, N, dtype=torch.int8, device="cuda")
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        crbm.sample(plan, psi, spins, 2, crbm.EXCHANGE, 11, 0, samples_out=out)
    want, ref = start.clone(), torch.zeros_like(out)
    crbm.sample(plan, psi, want, 2, crbm.EXCHANGE, 11, 0, samples_out=ref)
    for _ in range(3):
        spins.copy_(start)
        out.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, ref) and torch.equal(spins, want)
    plan.close()
