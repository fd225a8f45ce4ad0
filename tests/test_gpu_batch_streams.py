"""What the batch's stages write past the caches goes by the working set of the
chunk that runs together, not by the whole batch: the descriptors in the workspace
hold the choice (bit 0 the state and the register, bit 1 FP64 gradients).  Bytes of
a chunk: 3 x 5 doubles a node for two states and the register, 9 values for the
gradients; the lines lie at 288 and 512 MB.  On either side the batch gives the
bits of the instances run alone."""
import numpy as np
import pytest

from paper_1912_12059_amd import inputs as I

pytestmark = pytest.mark.gpu
PHYS = dict(T=0.85, eps=1e-3, kappa=1e-5, alpha=1000.0, beta=1e-3)


def _mesh(N, nel):
    return {"nel": nel, "N": N, "hi": tuple(n / nel[-1] for n in nel)}


def _streams(b, meshes):
    """Choice of every instance, from its descriptor: four pointers (state, its copy,
    register, gradients), four more of the mesh, its extents, elements, node stride,
    XCDs and the choice."""
    import torch

    w = b.work.view(-1)
    w = w[: w.numel() // 8 * 8].view(torch.int64).cpu().numpy()
    out = []
    for i, m in enumerate(meshes):
        off = 8 * b.view(i).storage_offset()
        at = np.flatnonzero((w[:-11] == b.U.data_ptr() + off) & (w[2:-9] == b.dU.data_ptr() + off))
        assert len(at) == 1, (i, at)
        d = w[at[0]: at[0] + 12].view(np.int32)
        assert tuple(d[16:20]) == m["nel"] + (int(np.prod(m["nel"])),)
        out.append(int(d[23]))
    return out


# meshes of 256 MB (FP64, N = 4), 192 MB (FP64, N = 3) and 208 MB (mixed, N = 4) each
CASES = [
    ("one group, one chunk", [_mesh(4, (22, 22, 22))] * 3, 0, [(0, [0, 0])], [3, 3, 3]),
    ("one group, a chunk each", [_mesh(4, (22, 22, 22))] * 3, 0, [(0, [0, 256])], [0, 0, 0]),
    ("one group, a chunk each, persistent grid", [_mesh(4, (22, 22, 22))] * 3, 0, [(0, [2, 256])], [0, 0, 0]),
    ("two groups, each below the line", [_mesh(4, (22, 22, 22)), _mesh(3, (25, 25, 25))], 0, [], [0, 0]),
    ("chunks of two and one", [_mesh(3, (25, 25, 25))] * 3, 0, [(0, [2, 400])], [1, 1, 0]),
    ("mixed, two in a chunk", [_mesh(4, (22, 22, 22))] * 2, 1, [(0, [0, 0])], [1, 1]),
    ("mixed, a chunk each", [_mesh(4, (22, 22, 22))] * 2, 1, [(0, [0, 200])], [0, 0]),
]


@pytest.mark.parametrize("what,meshes,precision,groups,expected", CASES, ids=[c[0] for c in CASES])
def test_chunks_stream_by_their_own_bytes(gpu, what, meshes, precision, groups, expected):
    import torch

    b = gpu.Batch(meshes, precision=precision, **PHYS)
    for g, (gridmul, mib) in groups:
        gpu.nsk_batch_set_group(b.b, g, 0, gridmul, 5, mib)
    assert _streams(b, meshes) == expected
    states = {}
    for m in meshes:
        key = (m["N"], m["nel"])
        if key not in states:
            states[key] = torch.from_numpy(I.smooth_random(3, m["N"], m["nel"], seed=9, hi=m["hi"])[1]).to("cuda:0")
    for i, m in enumerate(meshes):
        b.set_state(i, states[(m["N"], m["nel"])])
    dt = 1e-6
    b.rk_step(dt, 2)
    alone = {}
    for key, U in states.items():
        m = next(x for x in meshes if (x["N"], x["nel"]) == key)
        s = gpu.Solver(dim=3, N=m["N"], nel=m["nel"], hi=m["hi"], precision=precision, **PHYS)
        s.set_state(U)
        s.rk_step(dt, 2)
        alone[key] = s.get_state().clone().reshape(-1)
        s.close()
    for i, m in enumerate(meshes):
        assert torch.equal(b.get_state(i).reshape(-1), alone[(m["N"], m["nel"])]), (what, i)
    b.close()
