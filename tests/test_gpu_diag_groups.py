"""Diagnostics and the step size at the edges of the groups of whole elements
that a workgroup walks: fewer elements than one group holds, exactly one group,
one element more, and one element a direction (its own neighbour on both
sides).  kappa is large, so that the lifted gradient carries the energy.

The energy is a sum of at most 1e4 terms of size <= 1 + kappa |grad c|^2/2, each
formed to some ten roundings: 1e-12 of the sum of magnitudes, which is bounded
here by |E| plus twice the bound 4 |W| of the bulk term.  With the lifting in
FP32 the gradient carries the round-off of FP32 times (N+1)^2: 2e-5."""
import numpy as np
import pytest

from paper_1912_12059_amd import inputs as I

pytestmark = pytest.mark.gpu
PHYS = dict(T=0.85, eps=1e-3, kappa=1e-2)


def _meshes():
    for N in (1, 2, 3, 4, 5, 6):
        held = 256 // (N + 1)
        for nel in (1, held - 1, held, held + 1):
            yield 1, N, (nel,)
    for N in (1, 2, 4, 6):
        held = 256 // (N + 1) ** 2
        for nel in ((1, 1), (held, 1), (1, held + 1), (3, 5)):
            yield 2, N, nel
    for N in (1, 2, 3, 4, 5):
        held = 256 // (N + 1) ** 3
        for nel in ((1, 1, 1), (held, 1, 1), (1, held + 1, 1), (3, 2, 5)):
            yield 3, N, nel


@pytest.mark.parametrize("model,precision", [(0, 0), (0, 1), (1, 0)])
@pytest.mark.parametrize("dim", [1, 2, 3])
def test_diagnostics_groups(O, gpu, dim, model, precision):
    for d, N, nel in _meshes():
        if d != dim:
            continue
        m, U = I.smooth_random(dim, N, nel, seed=dim + N + sum(nel))
        kw = dict(PHYS) if model else dict(PHYS, alpha=500.0, beta=1e-3)
        if model:
            U, kw["model"] = np.ascontiguousarray(U[:-1]), 1
        one = (1,) * (3 - dim)
        P = O.Problem(dim=dim, N=N, nel=tuple(nel) + one, lo=tuple(m.lo) + (0.0,) * (3 - dim),
                      hi=tuple(m.hi) + (1.0,) * (3 - dim), xbreaks=m.xbreaks, **kw)
        s = gpu.Solver(dim=dim, N=N, nel=tuple(nel), lo=tuple(m.lo) + (0.0,) * 3, hi=tuple(m.hi) + (1.0,) * 3,
                       xbreaks=m.xbreaks, precision=precision, **(dict(kw, flux=2) if model else kw))
        s.set_state(U)
        got, ref = s.diagnostics(), O.diagnostics(P, s.get_state().cpu().numpy().reshape(U.shape))
        dt, dtr = s.dt_estimate(0.5), O.dt(P, U, 0.5)
        s.close()
        np.testing.assert_allclose(got["mass"], ref["mass"], rtol=1e-12, atol=1e-13, err_msg=str((N, nel)))
        for k in ("e_kin", "rho_min", "rho_max", "max_wavespeed"):
            assert got[k] == pytest.approx(ref[k], rel=1e-12), (k, N, nel)
        tol = 2e-5 if precision else 1e-12
        assert abs(got["e_total"] - ref["e_total"]) <= tol * (abs(ref["e_total"]) + 8.0), (N, nel)
        assert got["nonfinite"] == 0 and got["status"] == 0
        assert dt == pytest.approx(dtr, rel=1e-12), (N, nel)
