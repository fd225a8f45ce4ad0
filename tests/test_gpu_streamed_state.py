"""Stages whose arrays are too large for the last-level cache write them past it.
Meshes on both sides of either size limit, 2D and 3D, even and odd numbers of
nodes an element, FP64 and mixed precision: steps by the whole mesh against the
same steps with each stage's right-hand side from nsk_rhs, whose results are
always written through the caches.  The same kernel forms the right-hand side, so
that the states differ by the roundings of the update alone: two a stage, 1e-14 of
the largest value after ten stages.  In mixed precision those may flip an FP32
rounding of the right-hand side, 2^-24 of dt times its terms (below 1/10 of the
state here): 1e-8."""
import numpy as np
import pytest

from paper_1912_12059_amd import inputs as I

pytestmark = pytest.mark.gpu
PHYS = dict(T=0.85, eps=1e-3, kappa=1e-5, alpha=500.0, beta=1e-3)
A = (0.0, -567301805773.0 / 1357537059087.0, -2404267990393.0 / 2016746695238.0,
     -3550918686646.0 / 2091501179385.0, -1275806237668.0 / 842570457699.0)
B = (1432997174477.0 / 9575080441755.0, 5161836677717.0 / 13612068292357.0, 1720146321549.0 / 2090206949498.0,
     3134564353537.0 / 4481467310338.0, 2277821191437.0 / 14882151754819.0)


@pytest.mark.parametrize("dim,N,nel,precision", [
    (3, 4, (23, 23, 22), 0), (3, 4, (24, 23, 23), 0), (3, 4, (28, 28, 28), 0), (3, 3, (35, 35, 36), 0),
    (3, 4, (24, 24, 25), 1), (3, 4, (25, 25, 25), 1), (2, 4, (290, 290), 0), (2, 4, (295, 295), 0), (2, 5, (330, 330), 0),
])
def test_streamed_steps(gpu, dim, N, nel, precision):
    import torch

    m, U = I.smooth_random(dim, N, nel, seed=3)
    dt = 1e-3 / (max(nel) * (2 * N + 1) * 40.0)
    s = gpu.Solver(dim=dim, N=N, nel=nel, precision=precision, **PHYS)
    s.set_state(U)
    s.rk_step(dt, 2)
    got = s.get_state().clone()
    s.set_state(U)
    u = s.get_state().clone()
    du = torch.zeros_like(u)
    for k in range(10):
        r = s.rhs(u).reshape(u.shape)
        du = A[k % 5] * du + dt * r
        u = u + B[k % 5] * du
    s.close()
    assert torch.isfinite(got).all()
    for v in range(U.shape[0]):
        a, b = got.reshape(U.shape[0], -1)[v], u.reshape(U.shape[0], -1)[v]
        assert (a - b).abs().max() <= (1e-8 if precision else 1e-14) * b.abs().max(), v
