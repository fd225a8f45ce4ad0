"""Loss and gradient of the closure network at the edges of the training
kernel's tiles (128 samples, 32 a wave; more than 256 tiles are walked), against
plain torch in 64 bits with the same rounding points."""
import math

import numpy as np
import pytest

from paper_1912_12059_amd import closure as CL

pytestmark = pytest.mark.gpu

# A BF16 activation whose FP32 pre-activation differs from the 64-bit one in
# its last places may round the other way, which changes it by at most 2^-8 of
# itself; the gradient is linear in each activation, so it moves by no more
# than that, relative to its norm.  FP32 sums of 64 terms add 64 2^-24.
GRAD_TOL = 2.0 ** -8


def _bf16(x):
    import torch

    return x.to(torch.float32).to(torch.bfloat16).to(torch.float64)


def _reference(p, X, Y, q):
    import torch

    P, o = {}, 0
    for name, shape in CL.LAYOUT:
        k = math.prod(shape)
        P[name] = p[o:o + k].reshape(shape)
        o += k
    z1 = X @ P["W1"].T + P["b1"]
    h1 = _bf16(z1.clamp(min=0))
    z2 = h1 @ P["W2"].T + P["b2"]
    h2 = _bf16(z2.clamp(min=0))
    z3 = h2 @ P["W3"].T + P["b3"]
    h3 = z3.clamp(min=0)
    r = h3 @ P["W4"].T + P["b4"] - Y * torch.tensor(q, dtype=torch.float64, device=Y.device)
    dy = r / len(X)
    d3 = (dy @ P["W4"]) * (z3 > 0)
    d2 = (d3 @ P["W3"]) * (z2 > 0)
    d1 = (d2 @ P["W2"]) * (z1 > 0)
    g = [d1.T @ X, d1.sum(0), d2.T @ h1, d2.sum(0), d3.T @ h2, d3.sum(0), dy.T @ h3, dy.sum(0)]
    return 0.5 * float((r * r).sum()) / len(X), torch.cat([t.reshape(-1) for t in g])


@pytest.mark.parametrize("n", [1, 31, 33, 127, 128, 129, 1000, 32768, 32769, 70001])
def test_loss_grad_at_tile_edges(gpu, n):
    import torch

    g = np.random.Generator(np.random.PCG64(n))
    net = CL.Network(params=CL.init_params(3) + g.uniform(-0.05, 0.05, CL.NPARAM).astype(np.float32))
    pool = n + 17
    X = torch.from_numpy(g.normal(size=(pool, 4)).astype(np.float32)).cuda()
    Y = torch.from_numpy(g.normal(size=(pool, 2)).astype(np.float32)).cuda()
    idx = torch.from_numpy(g.integers(0, pool, size=n, dtype=np.int32)).cuda()
    q = (1.0, 0.5)
    loss, grad = net.loss_grad(X, Y, idx, tscale=q)
    p = torch.from_numpy(net.bf16_values()).cuda()
    lr, gr = _reference(p, X[idx.long()].double(), Y[idx.long()].double(), q)
    assert abs(float(loss) - lr) <= GRAD_TOL * lr
    assert float((grad.double() - gr).norm()) <= GRAD_TOL * float(gr.norm())
    # without a gather, and from addresses that are only aligned to a value
    sh = torch.empty(4 * n + 1, dtype=torch.float32, device="cuda")[1:].reshape(n, 4)
    sh.copy_(X[:n])
    st = torch.empty(2 * n + 1, dtype=torch.float32, device="cuda")[1:].reshape(n, 2)
    st.copy_(Y[:n])
    l0, g0 = net.loss_grad(X[:n], Y[:n], tscale=q)
    w = torch.empty(CL.NPARAM + 1, dtype=torch.int16, device="cuda")[1:]
    w.copy_(net.w)
    net.w = w
    l1, g1 = net.loss_grad(sh, st, tscale=q)
    assert torch.equal(l0, l1) and torch.equal(g0, g1)
