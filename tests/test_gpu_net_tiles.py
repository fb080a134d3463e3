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
