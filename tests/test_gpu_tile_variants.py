"""The launch shapes whose elements per workgroup differ (degrees 1 and 2 in 2D and
3D, 1D): right-hand sides and steps of both variants, in every element order, have
the same bits, on meshes that leave the last workgroup of either variant part empty,
and variant 1 meets the oracle."""
import numpy as np
import pytest

from paper_1912_12059_amd import inputs as I
from tolerances import RHS_ULPS, rhs_err_ulps, term_scales

pytestmark = pytest.mark.gpu
PHYS = dict(T=0.85, eps=1e-3, kappa=1e-5, alpha=500.0, beta=1e-3)
# elements per workgroup, variants 0 and 1: 3D 16, 8 and 7, 3 (N = 1, 2); 2D 32, 16
# and 21, 10; 1D N = 3 64, 32
MESHES = [(3, 1, (3, 3, 3)), (3, 1, (17, 1, 1)), (3, 2, (2, 2, 2)), (3, 2, (5, 3, 1)),
          (2, 1, (11, 3)), (2, 1, (7, 7)), (2, 2, (11, 2)), (2, 2, (5, 5)), (1, 3, (65,)), (1, 3, (97,))]
MODELS = {"fp64": dict(), "mixed": dict(precision=1), "hllc": dict(flux=1), "mixed hllc": dict(precision=1, flux=1),
          "nsk": dict(model=1, flux=2), "subcell": dict(subcell=1, subcell_threshold=-3.0),
          "subcell hllc": dict(subcell=1, subcell_threshold=-3.0, flux=1)}


@pytest.mark.parametrize("model", MODELS)
@pytest.mark.parametrize("dim,N,nel", MESHES)
def test_variants_same_bits(O, gpu, dim, N, nel, model):
    m, U = I.smooth_random(dim, N, nel, seed=3 + N)
    if model == "nsk":
        U = np.ascontiguousarray(U[: dim + 1])
    full = tuple(nel) + (1,) * (3 - dim)
    s = gpu.Solver(dim=dim, N=N, nel=full, hi=(1.0, 1.0, 1.0), **PHYS, **MODELS[model])
    ref = None
    for variant in (0, 1):
        for order in range(6):
            gpu.nsk_set_tile(s.ctx, variant, order)
            R = s.rhs(U).cpu().numpy()
            s.set_state(U)
            s.rk_step(1e-6, 3)
            out = (R, s.get_state().cpu().numpy())
            assert all(np.isfinite(x).all() for x in out)
            ref = ref or out
            assert all(np.array_equal(a, b) for a, b in zip(out, ref)), (variant, order)
    s.close()
    if model == "fp64":
        Rc = O.rhs(O.Problem(dim=dim, N=N, nel=full, lo=(0.0,) * 3, hi=(1.0,) * 3, **PHYS), U)
        assert rhs_err_ulps(R, Rc, term_scales(O, N, min(1.0 / n for n in nel), U, PHYS["alpha"])) <= RHS_ULPS


@pytest.mark.parametrize("dim,N,nel,rep", [(3, 4, (14, 14, 14), (2, 2, 2)), (3, 3, (18, 18, 17), (2, 2, 2)),
                                           (2, 4, (200, 200), (3, 3)), (2, 5, (165, 165), (3, 3))])
def test_gradients_past_the_caches(gpu, dim, N, nel, rep):
    """FP64 gradients are written past the caches above 512 MB of state and gradients: the
    right-hand side of a mesh above against that of the periodic mesh it repeats, which
    is below (elements of edge 1/4 in both: the same values), bit for bit."""
    import torch

    m, U = I.smooth_random(dim, N, nel, seed=4)
    nn = (N + 1) ** dim
    u = torch.from_numpy(U).to("cuda:0").reshape((len(U),) + tuple(reversed(nel)) + (nn,))
    values = 3 * len(U) + dim * (dim + 1) // 2 + dim
    out = []
    for r in ((1,) * dim, rep):
        n = tuple(a * b for a, b in zip(nel, r))
        assert (8 * values * nn * np.prod(n) > 512e6) == (r == rep)
        s = gpu.Solver(dim=dim, N=N, nel=n + (1,) * (3 - dim), hi=tuple(0.25 * k for k in n) + (1.0,) * (3 - dim), **PHYS)
        R = s.rhs(u.repeat((1,) + tuple(reversed(r)) + (1,)).reshape(len(U), -1, nn).contiguous()).clone()
        out.append(R.reshape((len(U),) + tuple(reversed(n)) + (nn,)))
        s.close()
    assert torch.equal(out[0].repeat((1,) + tuple(reversed(rep)) + (1,)), out[1])
