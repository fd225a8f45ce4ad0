"""Launches whose element lines take two lanes each (small ones from degree 4 in 2D,
degree 4 in 3D) against launches with one lane a line: a periodic mesh and the same
one repeated until it is too large for the first form, on elements of the same
extent, so that both form the same values.  The forms do the same operations in the
same order: same bits.  One element, one workgroup's elements, one more, ragged
ones; Rusanov and HLLC, mixed precision and the original NSK equations."""
import pytest

from paper_1912_12059_amd import inputs as I

pytestmark = pytest.mark.gpu
PHYS = dict(T=0.85, eps=1e-3, kappa=1e-5, alpha=500.0, beta=1e-3)
# the large meshes are above 6144, 20480 and 24576 elements (2D, N = 4, 5, 6) and 1024 (3D)
MESHES = [(2, 4, (1, 1), (103, 103)), (2, 4, (6, 1), (42, 42)), (2, 4, (7, 5), (18, 18)), (2, 4, (64, 24), (3, 3)),
          (2, 5, (1, 1), (176, 176)), (2, 5, (5, 1), (79, 79)), (2, 5, (3, 7), (39, 39)),
          (2, 6, (1, 1), (157, 157)), (2, 6, (4, 1), (79, 79)), (2, 6, (5, 3), (41, 41)),
          (3, 4, (1, 1, 1), (11, 11, 11)), (3, 4, (2, 1, 1), (9, 9, 9)), (3, 4, (5, 3, 2), (4, 4, 3))]


@pytest.mark.parametrize("precision,flux,model", [(0, 0, 0), (1, 0, 0), (0, 1, 0), (1, 1, 0), (0, 2, 1)])
@pytest.mark.parametrize("dim,N,nel,rep", MESHES)
def test_same_bits_as_one_lane_a_line(gpu, dim, N, nel, rep, precision, flux, model):
    import torch

    m, U = I.smooth_random(dim, N, nel, seed=11 + N)
    if model == 1:
        U = U[: dim + 1]
    u = torch.from_numpy(U).to("cuda:0").reshape((len(U),) + tuple(reversed(nel)) + ((N + 1) ** dim,))
    out = []
    for r in ((1,) * dim, rep):
        n = tuple(a * b for a, b in zip(nel, r))
        one = (1,) * (3 - dim)
        s = gpu.Solver(dim=dim, N=N, nel=n + one, hi=tuple(0.25 * k for k in n) + (1.0,) * (3 - dim),
                       precision=precision, flux=flux, model=model, **PHYS)
        s.set_state(u.repeat((1,) + tuple(reversed(r)) + (1,)).reshape(len(U), -1, (N + 1) ** dim).contiguous())
        R = s.rhs(s.get_state()).clone()
        s.rk_step(2e-6, 3)
        out.append([x.reshape((len(U),) + tuple(reversed(n)) + (-1,)) for x in (R, s.get_state().clone())])
        s.close()
    for small, large in zip(*out):
        assert torch.isfinite(small).all()
        assert torch.equal(small.repeat((1,) + tuple(reversed(rep)) + (1,)), large)
