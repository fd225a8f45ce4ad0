"""HLLC in 3D with every side of its case distinction: velocities of several
times the sound speed in both directions (the flux of one side alone) and small
ones (the star region), each degree, FP64 and mixed precision.  Against the
oracle at the right-hand-side bounds of tests/tolerances.py."""
import numpy as np
import pytest

from paper_1912_12059_amd import inputs as I
from tolerances import MIXED_ULPS, RHS_ULPS, record, rhs_err_ulps, term_scales

pytestmark = pytest.mark.gpu
PHYS = dict(T=0.85, eps=1e-3, kappa=1e-5, alpha=500.0, beta=1e-3)


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("vmax", [0.5, 120.0])
@pytest.mark.parametrize("N", [1, 2, 3, 4, 5])
def test_hllc_branches(O, gpu, N, vmax, precision):
    nel = (3, 2, 2)
    m, U = I.smooth_random(3, N, nel, seed=40 + N, vmax=vmax)
    for diss_c in (0, 1):
        kw = dict(PHYS, flux=1, diss_c=diss_c)
        s = gpu.Solver(dim=3, N=N, nel=nel, hi=(1.0, 1.0, 1.0), precision=precision, **kw)
        R = s.rhs(U).cpu().numpy()
        s.close()
        Rc = O.rhs(O.Problem(dim=3, N=N, nel=nel, lo=(0.0,) * 3, hi=(1.0,) * 3, **kw), U)
        scales = term_scales(O, N, 1.0 / max(nel), U, PHYS["alpha"])
        if precision == 0:
            assert rhs_err_ulps(R, Rc, scales) <= RHS_ULPS
        else:
            err = np.abs(R - Rc).reshape(U.shape[0], -1).max(axis=1) / (2.0 ** -24 * scales)
            record("mixed rhs, FP32 ulps of term scale", err.max(), MIXED_ULPS)
            assert err.max() <= MIXED_ULPS, err
