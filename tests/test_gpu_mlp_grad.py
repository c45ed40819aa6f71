"""The training gradient at the edges of its tiles against the same arithmetic
on the CPU: BF16 weights, activations and deltas with FP64 sums.

A BF16 value may round to its neighbour where the device's FP32 sum lies on the
other side of a tie, which moves that factor of a term by 2^-8 and, through the
layers that follow, the terms made from it by no more; every term of a gradient
entry has two such factors and a tie is rare.  Bar: 2^-7 of the sum of the
entry's absolute terms; the loss, a sum of squares, to 2^-7.
"""
import ctypes as C

import numpy as np
import pytest

from oracle import mlp

pytestmark = pytest.mark.gpu


def _bf(a):
    u = np.ascontiguousarray(a, np.float32).view(np.uint32)
    u = (u + np.uint32(0x7fff) + ((u >> np.uint32(16)) & np.uint32(1))) & np.uint32(0xffff0000)
    return u.view(np.float32).astype(np.float64)


def _emulated(theta, X, T):
    """Gradient, loss, and the sums of absolute terms."""
    p = mlp.unpack(np.asarray(theta, np.float32).astype(np.float64))
    W1, W2, W3, W4 = _bf(p["W1"]), _bf(p["W2"]), _bf(p["W3"]), _bf(p["W4"]).ravel()
    n = X.shape[0]
    z1 = X @ W1.T + p["b1"]
    h1 = _bf(np.maximum(z1, 0))
    z2 = h1 @ W2.T + p["b2"]
    h2 = _bf(np.maximum(z2, 0))
    z3 = h2 @ W3.T + p["b3"]
    h3 = np.maximum(z3, 0)
    r = h3 @ W4 + p["b4"].ravel()[0] - T
    dy = (2.0 / n * r)[:, None]
    d3 = _bf(np.where(z3 > 0, dy * W4, 0))
    d2 = _bf(np.where(z2 > 0, d3 @ W3, 0))
    d1 = _bf(np.where(z1 > 0, d2 @ W2, 0))
    one = np.ones((n, 1))
    pairs = [(d1, _bf(X)), (d1, one), (d2, h1), (d2, one), (d3, h2), (d3, one),
             (_bf(dy), _bf(h3)), (_bf(dy), one)]
    g = np.concatenate([(a.T @ b).ravel() for a, b in pairs])
    size = np.concatenate([(abs(a).T @ abs(b)).ravel() for a, b in pairs])
    return g, (r * r).mean(), size


# one sample; a tile less one, whole, and one more; 256 workgroups' last tile
# ragged; two tiles in some workgroups; 512 workgroups, the last with one tile
@pytest.mark.parametrize("n", [1, 31, 32, 33, 8191, 8225, 65505, 65536 + 32])
def test_gradient_matches_emulation(n):
    import torch
    from paper_2510_12011_amd import _lib as L, sim
    ctx = sim.Simulation(0)
    rng = np.random.default_rng(n)
    theta = mlp.init_params(9).astype(np.float32)
    theta[-1] = 0.3
    X = rng.normal(size=(n, 4)).astype(np.float32)
    T = (np.sin(X[:, 0]) + X[:, 1] * X[:, 2]).astype(np.float32)
    ref, loss_ref, size = _emulated(theta, X.astype(np.float64), T.astype(np.float64))
    P, Xd, Td = (torch.from_numpy(a).cuda() for a in (theta, X, T))
    ptr = lambda t: C.c_void_p(t.data_ptr())
    nb = L.lib().mdx_mlp_grad_scratch(n)
    scratch = torch.empty(nb // 4, dtype=torch.float32, device="cuda:0")
    g = torch.full((mlp.N_PARAM,), np.nan, dtype=torch.float32, device="cuda:0")
    loss = torch.zeros(1, device="cuda:0")
    ctx._check(L.lib().mdx_mlp_grad(ctx._h, ptr(P), n, ptr(Xd), ptr(Td), ptr(g), ptr(loss),
                                    ptr(scratch), nb))
    g2 = torch.empty_like(g)
    ctx._check(L.lib().mdx_mlp_grad_noalloc(ctx._h, ptr(P), n, ptr(Xd), ptr(Td), ptr(g2), None))
    torch.cuda.synchronize()
    assert loss.item() == pytest.approx(loss_ref, rel=2.0 ** -7)
    assert (abs(g.cpu().numpy() - ref) <= 2.0 ** -7 * size + 1e-30).all()
    if n < 65505:
        assert torch.equal(g, g2)
