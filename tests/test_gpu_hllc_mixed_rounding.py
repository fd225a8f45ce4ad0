"""HLLC in mixed precision: how the two wave speeds are rounded is part of the
result.  SL = v - a comes from unrounded products v = m / rho, SR = v + a from rounded
ones; any other choice changes the FP32 flux at about one face in a thousand, by one
unit in the last place, and through the contraction 1e-5 and more of a node's rate.
The values below are right-hand sides at such nodes (variable, node, rate), a form of
the kernels each: 1D, two lanes a line, a lane a line, staged neighbours."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

RATES = [
    (1, 2, (3000,), [(1, 7273, -13055.97297220022), (1, 7272, 117063.7767937154), (1, 7270, 63543.49626409356)]),
    (2, 1, (60, 41), [(1, 4841, -224.58737933622803), (1, 1351, -250.93137420952795),
                      (1, 4837, -510.81454052781635)]),
    (2, 4, (26, 23), [(1, 3237, 45.63780487087777), (1, 4644, 402.7889367705363), (1, 4545, 854.187818725974)]),
    (3, 2, (9, 8, 7), [(1, 10025, -0.5430904704835979), (3, 1781, -0.6323641914655488),
                       (2, 6123, 1.886555932196161)]),
    (3, 4, (15, 14, 13), [(1, 193382, -0.08936690116634309), (1, 91695, 1.032150929555748),
                          (2, 125247, -5.599750464335578)]),
    (3, 5, (9, 8, 9), [(1, 38850, -0.9807120742804067), (1, 10798, 1.0980619234871338),
                       (2, 23495, -1.1915532103507562)]),
]


@pytest.mark.parametrize("dim, N, nel, rates", RATES, ids=["%dd-%d" % c[:2] for c in RATES])
def test_hllc_mixed_rates(gpu, dim, N, nel, rates):
    n = int(np.prod(nel)) * (N + 1) ** dim
    r = np.random.Generator(np.random.PCG64(7))
    U = np.empty((dim + 2, n))
    U[0] = 1.0 + 0.4 * r.random(n)
    for d in range(dim):
        U[1 + d] = U[0] * (0.2 * r.random(n) - 0.1)
    U[dim + 1] = U[0] + 0.01 * r.random(n)
    s = gpu.Solver(dim=dim, N=N, nel=nel, alpha=500.0, beta=1e-3, eps=1e-3, kappa=1e-5, precision=1, flux=1)
    R = s.rhs(U.reshape(-1)).cpu().numpy().reshape(dim + 2, -1)
    s.close()
    # what is left beside the FP32 values is their sum with FP64 sources
    for v, node, rate in rates:
        assert abs(R[v, node] - rate) <= 1e-9 * np.abs(R[v]).max(), (v, node, R[v, node])
