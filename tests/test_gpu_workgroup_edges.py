"""Right-hand sides on meshes at the edges of the kernels' workgroups: one
element, an element that is its own neighbour along some direction, exactly
the elements one workgroup holds, one fewer and one more.  Against the oracle,
at the right-hand-side bounds of tests/tolerances.py."""
import numpy as np
import pytest

from paper_1912_12059_amd import inputs as I
from tolerances import MIXED_ULPS, RHS_ULPS, rhs_err_ulps, record, term_scales

pytestmark = pytest.mark.gpu
PHYS = dict(T=0.85, eps=1e-3, kappa=1e-5, alpha=500.0, beta=1e-3)

# elements per workgroup: 3D 16, 7, 4, 2, 1 (N = 1..5), 2D 32, 21, 16, 9, 7, 5
# (N = 1..6), 1D 64 (N = 3) and 36 (N = 6)
MESHES = [(3, 1, (5, 3, 1)), (3, 1, (16, 1, 1)), (3, 2, (7, 1, 1)), (3, 2, (2, 2, 2)), (3, 3, (1, 1, 5)),
          (3, 3, (1, 2, 2)), (3, 4, (1, 1, 1)), (3, 4, (3, 1, 1)), (3, 4, (1, 2, 1)), (3, 5, (1, 1, 1)),
          (3, 5, (1, 2, 3)),
          (2, 1, (11, 3)), (2, 2, (21, 1)), (2, 3, (1, 17)), (2, 4, (1, 1)), (2, 4, (9, 1)), (2, 4, (5, 2)),
          (2, 5, (2, 3)), (2, 5, (1, 8)), (2, 6, (5, 1)), (2, 6, (2, 3)),
          (1, 3, (1,)), (1, 3, (64,)), (1, 3, (65,)), (1, 6, (37,))]


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("dim,N,nel", MESHES)
def test_rhs_at_workgroup_edges(O, gpu, dim, N, nel, precision):
    m, U = I.smooth_random(dim, N, nel, seed=5 + 7 * dim + N)
    full = tuple(nel) + (1,) * (3 - dim)
    s = gpu.Solver(dim=dim, N=N, nel=full, hi=(1.0, 1.0, 1.0), precision=precision, **PHYS)
    R = s.rhs(U).cpu().numpy()
    s.close()
    Rc = O.rhs(O.Problem(dim=dim, N=N, nel=full, lo=(0.0,) * 3, hi=(1.0,) * 3, **PHYS), U)
    scales = term_scales(O, N, min(1.0 / n for n in nel), U, PHYS["alpha"])
    if precision == 0:
        assert rhs_err_ulps(R, Rc, scales) <= RHS_ULPS
    else:
        err = np.abs(R - Rc).reshape(U.shape[0], -1).max(axis=1) / (2.0 ** -24 * scales)
        record("mixed rhs, FP32 ulps of term scale", err.max(), MIXED_ULPS)
        assert err.max() <= MIXED_ULPS, err
