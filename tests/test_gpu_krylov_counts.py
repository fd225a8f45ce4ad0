"""Implicit steps at Krylov spaces of one vector, of exactly one launch of basis
vectors (8), one more, and several launches, FP64 and FP32 basis, with and
without the source preconditioner and with projections never repeated, against
the oracle's dense Newton solves.  Stages are solved to 1e-13 of |B|, so that the
states agree to 1e-9 of each variable's largest value, as for any other count."""
import numpy as np
import pytest

from oracle import esdirk as E
from paper_1912_12059_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precond,basis_fp32,reorth_tol", [(0, 0, 0.5), (1, 0, 0.5), (1, 1, 0.5), (0, 1, 0.0)])
@pytest.mark.parametrize("gmres_m,factor", [(1, 0.1), (8, 20.0), (9, 20.0), (33, 20.0)])
def test_krylov_counts(O, gpu, gmres_m, factor, precond, basis_fp32, reorth_tol):
    m, U = I.smooth_random(1, 2, (11,), seed=6, rho_range=(1.6, 1.9), dc=0.0)
    kw = dict(eps=1e-2, kappa=1e-4, alpha=500.0, beta=1e-3)
    P = O.Problem(dim=1, N=2, nel=(11, 1, 1), lo=tuple(m.lo) + (0.0,) * 2, hi=tuple(m.hi) + (1.0,) * 2,
                  xbreaks=m.xbreaks, **kw)
    dt = factor * O.dt(P, U, 0.5)
    ref = E.run(P, U, dt, 2)
    s = gpu.Solver(dim=1, N=2, nel=(11,), lo=tuple(m.lo) + (0.0,) * 3, hi=tuple(m.hi) + (1.0,) * 3,
                   xbreaks=m.xbreaks, **kw)
    s.set_state(U)
    st = s.esdirk_step(dt, 2, newton_tol=1e-13, newton_max=200, gmres_rtol=1e-8, gmres_m=gmres_m, precond=precond,
                       basis_fp32=basis_fp32, reorth_tol=reorth_tol)
    got = s.get_state().cpu().numpy().reshape(ref.shape)
    s.close()
    assert st["converged"] == 1 and st["steps"] == 2
    assert st["gmres_iters"] <= gmres_m * st["newton_iters"]
    for v in range(ref.shape[0]):
        assert np.abs(got[v] - ref[v]).max() <= 1e-9 * max(np.abs(ref[v]).max(), 1e-300), v
