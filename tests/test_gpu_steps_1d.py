"""Whole Runge-Kutta steps in one launch on 1D meshes: exactly the elements a
workgroup holds (512 nodes), one fewer and one more, where ranges overlap, a
last range of one element, and meshes hardly larger than one range.  Bit for
bit against the same steps taken stage by stage (second tile variant)."""
import numpy as np
import pytest

from paper_1912_12059_amd import inputs as I

pytestmark = pytest.mark.gpu
PHYS = dict(T=0.85, eps=1e-3, kappa=1e-5, alpha=500.0, beta=1e-3)


def _sizes(N):
    held = 512 // (N + 1)
    own = held - 20
    return [1, 3, held - 1, held, held + 1, 2 * own, 2 * own + 1, 3 * own - 1]


@pytest.mark.parametrize("precision,flux", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("N", [1, 2, 3, 4, 5, 6])
def test_whole_steps_equal_stages(gpu, N, precision, flux):
    import torch

    for nel in _sizes(N):
        m, U = I.smooth_random(1, N, (nel,), seed=N + nel)
        dt = 1e-3 / (nel * (2 * N + 1) * 40.0)
        out = []
        for tile in (0, 1):
            s = gpu.Solver(dim=1, N=N, nel=(nel,), precision=precision, flux=flux, stream=torch.cuda.Stream(), **PHYS)
            gpu.nsk_set_tile(s.ctx, tile, 0)
            s.set_state(U)
            s.rk_step(dt, 1)   # one launch, or stage by stage
            s.rk_step(dt, 4)   # pairs of steps as a captured graph
            s.rk_step(dt, 3)
            state = s.get_state().cpu().numpy()
            out.append((state, s.dU.cpu().numpy()))
            s.close()
        assert np.isfinite(out[0][0]).all() and not np.array_equal(out[0][0], U)
        assert np.array_equal(out[0][0], out[1][0]), nel
        assert np.array_equal(out[0][1], out[1][1]), nel
