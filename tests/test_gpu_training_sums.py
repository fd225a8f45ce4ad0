"""Precision of the closure network's gradient: parameters and features are small
dyadic numbers, so that every pre-activation is exact in FP32 and rounds the same
way in 64 bits, and what is left is the rounding of the backward pass and of its
sums.  The bound is 2^-24 of the sum of the terms' magnitudes, element by element,
times the FP32 roundings on the way of a term: 2 of dy, 2 of dz3, 12 matrix steps of
dz2, 12 of dz1, 24 of a weight's sum over a tile (or 32 additions and 4 of a vector
sum), 2 of what a workgroup writes and of the result; 64 in all."""
import math

import numpy as np
import pytest

from paper_1912_12059_amd import closure as CL

pytestmark = pytest.mark.gpu
ROUNDINGS = 64
TILE, GRID = 128, 256  # samples of a tile, workgroups


def _dyadic(g, shape, bits, scale):
    return g.integers(-(2 ** bits) + 1, 2 ** bits, size=shape) * scale


def _params(g):
    """Weights of 3 bits: z1 multiples of 1/64, z2 of 2^-9, z3 of 2^-12 or coarser, all
    below 2^10, the outputs multiples of 2^-15."""
    out = [_dyadic(g, (64, 4), 3, 1 / 8), _dyadic(g, 64, 3, 1 / 8), _dyadic(g, (64, 64), 3, 1 / 32),
           _dyadic(g, 64, 3, 1 / 8), _dyadic(g, (64, 64), 3, 1 / 32), _dyadic(g, 64, 3, 1 / 8),
           _dyadic(g, (2, 64), 2, 1 / 16), _dyadic(g, 2, 3, 1 / 8)]
    return np.concatenate([a.ravel() for a in out]).astype(np.float32)


def _unpack(p):
    P, o = {}, 0
    for name, shape in CL.LAYOUT:
        k = math.prod(shape)
        P[name] = p[o:o + k].reshape(shape)
        o += k
    return P


def _forward(P, X):
    import torch

    bf = lambda x: x.to(torch.float32).to(torch.bfloat16).to(torch.float64)  # noqa: E731
    z1 = X @ P["W1"].T + P["b1"]
    h1 = bf(z1.clamp(min=0))
    z2 = h1 @ P["W2"].T + P["b2"]
    h2 = bf(z2.clamp(min=0))
    z3 = h2 @ P["W3"].T + P["b3"]
    for z in (z1, z2, z3):
        assert torch.equal(z, z.float().double())  # exact
    return z1, h1, z2, h2, z3, z3.clamp(min=0)


def _reference(P, X, Y, count):
    """Loss, gradient and the sums of their terms' magnitudes in 64 bits, row s of X
    and Y taken count[s] times."""
    import torch

    z1, h1, z2, h2, z3, h3 = _forward(P, X)
    r = h3 @ P["W4"].T + P["b4"] - Y
    n = float(count.sum())
    c = count[:, None]
    dy = r / n
    d3 = (dy @ P["W4"]) * (z3 > 0)
    d2 = (d3 @ P["W3"]) * (z2 > 0)
    d1 = (d2 @ P["W2"]) * (z1 > 0)
    # magnitudes: a rounding of dz at any layer goes through absolute products
    a3 = (dy.abs() @ P["W4"].abs()) * (z3 > 0)
    a2 = (a3 @ P["W3"].abs()) * (z2 > 0)
    a1 = (a2 @ P["W2"].abs()) * (z1 > 0)
    out = []
    for e3, e2, e1, ey, x in ((d3, d2, d1, dy, X), (a3, a2, a1, dy.abs(), X.abs())):
        g = [(c * e1).T @ x, (c * e1).sum(0), (c * e2).T @ h1, (c * e2).sum(0), (c * e3).T @ h2, (c * e3).sum(0),
             (c * ey).T @ h3, (c * ey).sum(0)]
        out.append(torch.cat([t.reshape(-1) for t in g]))
    return 0.5 * float((c * r * r).sum()) / n, out[0], out[1]


def _problem(seed, pool):
    import torch

    g = np.random.Generator(np.random.PCG64(seed))
    net = CL.Network(params=_params(g))
    P = _unpack(torch.from_numpy(net.bf16_values()).cuda())
    X = torch.from_numpy(_dyadic(g, (pool, 4), 3, 1 / 8)).cuda()
    h3 = _forward(P, X)[-1]
    y = h3 @ P["W4"].T + P["b4"]
    return net, P, X, y, g


def _check(net, P, X, Y, idx):
    import torch

    loss, grad = net.loss_grad(X.float(), Y.float(), idx)
    count = torch.bincount(idx.long(), minlength=len(X)).double()
    lr, gr, mag = _reference(P, X, Y.float().double(), count)
    bad = (grad.double() - gr).abs() > ROUNDINGS * 2.0 ** -24 * mag
    worst = float(((grad.double() - gr).abs() / (2.0 ** -24 * mag).clamp(min=1e-300)).max())
    assert not bad.any(), (int(bad.sum()), worst)
    assert abs(float(loss) - lr) <= ROUNDINGS * 2.0 ** -24 * lr


@pytest.mark.parametrize("n", [1, 127, 129, 1000, 32768, 32769])
def test_gradient_is_fp32(gpu, n):
    """Every term of dz counts: without its third part a sample's gradient is 2^-17 to
    2^-16 off, 128 to 256 of the roundings above."""
    import torch

    net, P, X, y, g = _problem(n, 257)
    Y = y + torch.from_numpy(_dyadic(g, (257, 2), 20, 2.0 ** -18)).cuda()
    _check(net, P, X, Y, torch.from_numpy(g.integers(0, 257, size=n, dtype=np.int32)).cuda())


def test_sums_over_tiles_keep_small_terms(gpu):
    """A workgroup's first tile has residuals of 1, its 31 others of 2^-22: what a matrix
    step of those adds is below half an ulp of the sum so far, and all of it is 31/4 2^-20
    of the result, 124 roundings."""
    import torch

    net, P, X, y, g = _problem(7, 2 * TILE)
    big = (torch.arange(2 * TILE, device="cuda") < TILE).double()[:, None]
    Y = y - torch.where(big > 0, 1.0, 2.0 ** -22)
    row = torch.arange(TILE, dtype=torch.int32, device="cuda")
    idx = torch.cat([row.repeat(GRID), (TILE + row).repeat(31 * GRID)])
    _check(net, P, X, Y, idx)


@pytest.mark.parametrize("n", [GRID * TILE + 5, 2 * GRID * TILE + TILE])
def test_last_tile_counts(gpu, n):
    """Residuals of 1 in the last tile, of 2^-22 in all before it."""
    import torch

    net, P, X, y, g = _problem(8, 2 * TILE)
    big = (torch.arange(2 * TILE, device="cuda") < TILE).double()[:, None]
    Y = y - torch.where(big > 0, 1.0, 2.0 ** -22)
    idx = torch.from_numpy(g.integers(TILE, 2 * TILE, size=n, dtype=np.int32)).cuda()
    last = (n - 1) // TILE * TILE
    idx[last:] -= TILE
    _check(net, P, X, Y, idx)


@pytest.mark.parametrize("target", [math.inf, -math.inf, math.nan])
@pytest.mark.parametrize("n", [1, 300])
def test_infinite_and_nan_targets(gpu, target, n):
    """One sample's target is not finite: the gradient is infinite, NaN and finite where
    the products of the plain formula are."""
    import torch

    net, P, X, y, g = _problem(9, n)
    Y = y - 0.5
    Y[n // 2, 0] = target
    idx = torch.arange(n, dtype=torch.int32, device="cuda")
    loss, grad = net.loss_grad(X.float(), Y.float(), idx)
    z1, h1, z2, h2, z3, h3 = _forward(P, X)
    dy = (h3 @ P["W4"].T + P["b4"] - Y) / n
    d3 = (dy[:, :, None] * P["W4"][None]).sum(1) * (z3 > 0)
    outer = lambda d, h: (d[:, :, None] * h[:, None, :]).sum(0)  # noqa: E731
    d2 = (d3[:, :, None] * P["W3"][None]).sum(1) * (z2 > 0)
    d1 = (d2[:, :, None] * P["W2"][None]).sum(1) * (z1 > 0)
    ref = torch.cat([t.reshape(-1) for t in (outer(d1, X), d1.sum(0), outer(d2, h1), d2.sum(0), outer(d3, h2), d3.sum(0),
                                             outer(dy, h3), dy.sum(0))])
    assert not math.isfinite(float(loss))
    assert torch.equal(grad.isnan(), ref.isnan())
    assert torch.equal(grad.isposinf(), ref.isposinf()) and torch.equal(grad.isneginf(), ref.isneginf())


def test_largest_values_stay_finite(gpu):
    """dz of 3.4e38, which rounds to infinity in BF16: the gradients that are finite stay so."""
    import torch

    net, P, X, y, g = _problem(10, 1)
    Y = y.clone()
    w4 = float(P["W4"][0].abs().max())
    Y[0, 0] = -3.4e38 / w4 if w4 > 1 else -3.4e38
    P["W4"][:] = 0.0
    P["W4"][0] = 1.0
    P["W3"][:] = 0.0
    P["W3"][:, 0] = 2.0 ** -7
    p = torch.cat([P[k].reshape(-1) for k, _ in CL.LAYOUT]).cpu().numpy().astype(np.float32)
    net = CL.Network(params=p)
    z1, h1, z2, h2, z3, h3 = _forward(P, X)
    dy = (h3 @ P["W4"].T + P["b4"] - Y).float().double()
    d3 = (dy @ P["W4"]) * (z3 > 0)
    assert float(d3.abs().max()) > 3.395e38
    loss, grad = net.loss_grad(X.float(), Y.float(), torch.zeros(1, dtype=torch.int32, device="cuda"))
    G = _unpack(grad.double())
    ref = d3.T @ h2
    ok = ref.abs() < 3.4e38
    assert ok.any() and (ref[ok] != 0).any()
    assert torch.isfinite(G["W3"][ok]).all() and torch.isfinite(G["b3"]).all()
    assert ((G["W3"] - ref).abs()[ok] <= ROUNDINGS * 2.0 ** -24 * ref.abs()[ok]).all()
    assert ((G["b3"] - d3[0]).abs() <= ROUNDINGS * 2.0 ** -24 * d3[0].abs()).all()
