"""The stopping test of the CG against the true residual, where one iteration takes nearly all of it away.

With a diagonal shift far above S the operator S + eps I is a multiple of the identity up to a relative spread of 1e-8:
one iteration lowers |r| by about that spread, two by its square.  The residual that the step reports, formed from the
solution in double, is then far below or far above the tolerance 1e-10, and the flag has to say which: a solve reported
converged is at or below the tolerance, one that ran out of iterations above it is flagged."""
import numpy as np
import pytest
import torch

import paper_2103_08804_amd as crbm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("solver,flags", [(crbm.CG_DENSE, crbm.PLAN_DENSE_S), (crbm.CG_MATFREE, 0)])
@pytest.mark.parametrize("N,M", [(4, 5), (11, 30)])
@pytest.mark.parametrize("maxit", [1, 2, 3, 50])
def test_reported_convergence_is_true(N, M, maxit, solver, flags):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    n, tol = 200, 1e-10
    r = np.random.default_rng(N + M)
    plan = crbm.Plan(crbm.CHAIN, N, 1, M, n, flags)
    seen = []
    for eps in np.geomspace(1e6, 1e10, 24):
        sig = (2 * r.integers(0, 2, size=(n, N)) - 1).astype(np.int8)
        T = (0.5 * (r.normal(size=(n, M)) + 1j * r.normal(size=(n, M)))).astype(np.complex64)
        R = (1 + 0.3 * r.normal(size=n) + 0.2j * r.normal(size=n)).astype(np.complex64)
        stats = torch.zeros(8, dtype=torch.float64, device="cuda")
        crbm.sr_step(plan, crbm.RBM.empty(N, M), torch.from_numpy(sig).cuda(), torch.from_numpy(T).cuda(),
                     torch.from_numpy(R).cuda(), 0.1, float(eps), solver, crbm.FP32, tol, maxit, stats)
        st = stats.cpu().numpy()
        seen.append((st[4], int(st[5]), int(st[6])))
    plan.close()
    print("residual, iterations, flags:", seen)
    for res, its, fl in seen:
        assert fl in (0, crbm.FLAG_NOT_CONVERGED)
        assert (fl == 0) == (res <= tol), (res, its, fl)
        assert 1 <= its <= maxit
        assert fl == 0 or maxit == 1     # the second iteration always reaches the tolerance here
