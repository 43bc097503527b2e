"""Log amplitude, local energy and tanh theta at the edges of their kernels, against the oracle.

The theta product reads spins as sign bits, 32 sites to a word and 128 rows to a tile: chains of 30 to 256 sites
around the word boundaries, row counts that leave partial tiles, rows that start at odd addresses.  The local
energy takes M in groups of 64 units.  Small phases, so no theta is next to
a zero of cosh, and 1e-5 relative holds as in the other estimator tests.  The second test has arbitrary phases and
wide M: samples next to a node take the double-precision form; its bounds are those of rounding theta."""
import numpy as np
import pytest
import synth
import torch

import paper_2103_08804_amd as crbm
from gpu_util import eloc_rounding_bound, logpsi_rounding_bound, np_of, rel_err, to_device_rbm, to_oracle_rbm, wrapped

pytestmark = pytest.mark.gpu
TOL = 1e-5


def _run(orc, N, M, sig, std, sim, shift):
    fit_d = to_device_rbm(orc.RBM(*synth.random_rbm_arrays(13 * N + M, N, M, std, std_im=sim)))
    n = sig.shape[0]
    raw = torch.zeros(n * N + shift, dtype=torch.int8, device="cuda")
    sig_d = raw[shift:].view(n, N)
    sig_d.copy_(torch.from_numpy(sig))
    plan = crbm.Plan(crbm.CHAIN, N, 1, M, n)
    lp = torch.zeros(n, dtype=torch.complex64, device="cuda")
    el = torch.zeros_like(lp)
    T = torch.zeros(n, M, dtype=torch.complex64, device="cuda")
    crbm.local_estimators(plan, fit_d, sig_d, logpsi_out=lp, eloc_out=el, tanh_out=T)
    torch.cuda.synchronize()
    plan.close()
    fit = to_oracle_rbm(orc, fit_d)
    lat = orc.Lattice(0, N)
    return fit, lat, [np_of(x).astype(np.complex128) for x in (lp, el, T)], orc.logpsi(fit, sig), \
        orc.local_energy(fit, lat, sig)


@pytest.mark.parametrize("N,M,n,shift", [
    (30, 192, 129, 0), (32, 193, 127, 1), (33, 256, 61, 0), (34, 257, 37, 3), (64, 448, 130, 1), (66, 449, 35, 0),
    (96, 512, 14, 2), (128, 65, 131, 0), (129, 320, 33, 1), (256, 384, 19, 1), (250, 33, 258, 0), (2, 200, 5, 1)])
def test_estimators_at_the_edges(orc, N, M, n, shift):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    sig = synth.random_spins(N + n, n, N, zero_magnetisation=(N % 2 == 0))
    fit, lat, (lp, el, T), lp_ref, el_ref = _run(orc, N, M, sig, 0.02, 0.01, shift)
    O_ref = orc.logderiv(fit, sig)
    assert np.max(np.abs(lp.real - lp_ref.real) / np.maximum(np.abs(lp_ref.real), 1.0)) < TOL
    assert np.max(np.abs(wrapped(lp.imag - lp_ref.imag))) < TOL * max(1.0, np.abs(lp_ref).max())
    assert rel_err(el, el_ref) < TOL
    assert rel_err(T, O_ref[:, N:N + M]) < TOL


@pytest.mark.parametrize("M", [200, 257, 449])
def test_wide_next_to_zeros(orc, M):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    sig = orc.enumerate_configs(10)
    fit, lat, (lp, el, _), lp_ref, el_ref = _run(orc, 10, M, sig, 0.1, 0.5, 0)
    th = fit.b[None, :] + sig.astype(np.float64) @ fit.W
    print("M", M, "smallest |cosh theta|", np.abs(np.cosh(th)).min())
    blp = logpsi_rounding_bound(fit, sig) + TOL * np.maximum(np.abs(lp_ref.real), 1.0)
    assert np.all(np.abs(lp.real - lp_ref.real) <= blp)
    bel = eloc_rounding_bound(fit, lat.bonds(), sig) + TOL * np.abs(el_ref).max()
    print("E_loc error over bound", (np.abs(el - el_ref) / bel).max())
    assert np.all(np.abs(el - el_ref) <= bel)
