"""Gradients of the network at grids where the kernels' tiles end (needs an MI355X): the weight
gradient takes 32 x 4 x (1, 2 or 4) voxel tiles at each of the three levels, so a side of the
finest grid below, at and just past a tile, and a ragged last tile at every level.

Same oracle and bars as the parity tests of test_gpu_net.py: both sides round the same
intermediates to BF16, so 1e-2 of the loss and 3e-2 of a gradient's 2-norm cover rounding
flips, and a voxel row or plane left out of a sum at these sizes is at least 1/36 of it.
"""
import numpy as np
import pytest

from oracle import conv as C
from test_gpu_net import bf16, ctx, from_flat, hf, rel, setup_net, torch, x16_of  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(4, 4, 4), (4, 8, 36), (20, 4, 32), (12, 20, 68)])
def test_gradients_at_tile_edges(ctx, shape):  # noqa: F811
    net, p = setup_net(ctx, seed=11)
    rng = np.random.default_rng(sum(shape))
    x3 = bf16(rng.standard_normal(shape + (3,)))
    t = rng.standard_normal(shape + (2,)).astype(np.float32)
    L = net.train_step(x16_of(x3), torch.from_numpy(t).cuda(), update=False)
    out, cache = C.forward(p, x3, q=bf16)
    Lref, dout = C.loss(out, t.astype(np.float64))
    g_ref, _ = C.backward(p, cache, dout, q=bf16)
    assert abs(L - Lref) <= 1e-2 * abs(Lref)
    g = from_flat(net.get_grads())
    for k in g_ref:
        assert rel(g[k], g_ref[k]) <= 3e-2, (k, rel(g[k], g_ref[k]))


def crop_of(t, corner, n):
    z, y, x = corner
    return t[z:z + n, y:y + n, x:x + n].contiguous()


def test_large_tiles_equal_small_tiles(ctx):  # noqa: F811
    """A (260, 264, 268) grid runs the convolutions' large tiles at all three levels, with a ragged
    last tile in every direction; a 60^3 cut of it runs the small ones.  Away from the cut's inner
    faces by more than the network's reach (24 voxels) both compute the same sums in the same
    order: equal bits.  The gradients of a loss that differs from zero in a 4^3 window only stay
    within the cut; they are scaled by the sum of squares of the target, whose rounding reaches
    every stored BF16 gradient: the bar of the parity tests, 3e-2."""
    shape, n = (260, 264, 268), 60
    net, _ = setup_net(ctx, seed=12)
    gen = torch.Generator("cuda").manual_seed(5)
    x = torch.zeros(shape + (16,), dtype=torch.bfloat16, device="cuda")
    x[..., :3] = torch.randn(shape + (3,), generator=gen, device="cuda").to(torch.bfloat16)
    out = net.eval(x)
    last = tuple(s - n for s in shape)
    mid = (100, 96, 120)
    for corner, a, b in (((0, 0, 0), 0, 32), (last, 28, 60), (mid, 28, 32)):
        got = net.eval(crop_of(x, corner, n))
        assert torch.equal(got[a:b, a:b, a:b], crop_of(out, corner, n)[a:b, a:b, a:b]), corner

    w = torch.randn((4, 4, 4, 2), generator=gen, device="cuda")
    grads = []
    for xx, oo, c in ((x, out, tuple(m + 28 for m in mid)), (crop_of(x, mid, n), None, (28, 28, 28))):
        t = (net.eval(xx) if oo is None else oo).clone()
        t[c[0]:c[0] + 4, c[1]:c[1] + 4, c[2]:c[2] + 4] += w
        net.train_step(xx, t, update=False)
        g = from_flat(net.get_grads())
        den = float((t.double() ** 2).sum())
        grads.append({k: v * den for k, v in g.items()})
    for k in grads[0]:
        assert rel(grads[0][k], grads[1][k]) <= 3e-2, (k, rel(grads[0][k], grads[1][k]))
