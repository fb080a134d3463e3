"""The spectral operator's own transforms on planes with a short side and on long z-columns (needs
an MI355X): lanes shared between butterflies for 2 to 32 lines along either axis (remainders of 64
among them), blocks of one to eight waves, 32 and 64 columns per block of the z pass.  In complex128
the lanes are shared for few vectors and not for many: a vector's product must not depend on how
many there are.  Bars: those of test_gpu_spectral.py.
"""
import numpy as np
import pytest

from test_gpu_spectral import (U32, ctx, dev, hf, host, inputs, make, spectral_apply_bound, torch)  # noqa: F401

pytestmark = pytest.mark.gpu

# (nz, ny, nx); 200, 300: 32 columns in complex64; 120, 98: in complex128
SHAPES = [(64, 4, 64), (6, 128, 4), (200, 20, 20), (300, 24, 28), (120, 16, 36), (98, 27, 15), (9, 64, 7), (12, 45, 32),
          (2, 16, 32), (36, 30, 9), (3, 250, 12), (64, 128, 2), (20, 10, 27)]


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("shape", SHAPES)
def test_products_on_thin_planes(ctx, shape, prec):  # noqa: F811
    o, g = make(ctx, shape, 31, 9.0)
    rng = np.random.default_rng(32)
    nv = max(8, -(-400 // shape[0]))  # more than 384 planes: in complex128 the other way to use lanes
    x = inputs(rng.standard_normal((nv,) + shape) + 1j * rng.standard_normal((nv,) + shape), prec)
    shift = -0.21 + 0.83j
    xd = dev(x).to(torch.complex128 if prec == "f64" else torch.complex64)
    many = hf.apply(g, xd, shift)
    alone = hf.apply(g, xd[:1].contiguous(), shift)
    assert torch.equal(alone[0], many[0])
    unit = 1.0 if prec == "f32" else 2.0 ** -53 / U32
    many = host(many)
    for k in (0, nv - 1):
        ref = o.apply(x[k], shift)
        bound = unit * spectral_apply_bound(x[k], float(o.lam.max()), o.kappa, o.damp, shift)
        assert np.abs(many[k] - ref).max() <= bound, (k, np.abs(many[k] - ref).max(), bound)


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("shape", [(30, 5, 60), (60, 48, 6), (128, 14, 18)])
def test_solves_on_thin_planes(ctx, shape, prec):  # noqa: F811
    # every option of a step (first with the residual, last adding y1, two outputs, one factor),
    # systems leaving the batch: against the same solve of the right-hand sides one by one, where
    # complex128 shares lanes throughout: same steps and the same bits
    o, g = make(ctx, shape, 33, 12.0)
    rng = np.random.default_rng(34)
    f = rng.standard_normal((4,) + shape) + 1j * rng.standard_normal((4,) + shape)
    f[2] *= 1e-2
    fd = dev(f).to(torch.complex128 if prec == "f64" else torch.complex64)
    for q in (1, 2, 5):
        cg = hf.Contour(g, 6, 1.0, 0.4, q)
        y, st = hf.shifted_solve(g, cg, fd, reduce=5.0, max_steps=40)
        for r in range(4):
            y1, s1 = hf.shifted_solve(g, cg, fd[r:r + 1].contiguous(), reduce=5.0, max_steps=40)
            assert np.array_equal(st[:, r], s1[:, 0]), (q, r)
            assert torch.equal(y[:, r], y1[:, 0]), (q, r)
