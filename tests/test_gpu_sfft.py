"""The spectral operator's own transforms (sides of prime factors up to 7; needs an MI355X): every
radix as first, middle and last stage, sides with one stage, planes of less and of more than 64
points a side, both precisions, and the factor in the last pass for every option of a step.

Bars: those of test_gpu_spectral.py (10 u log2 N of the largest eigenvalue for a product, holding
for any order of radix-2 to radix-8 stages), one system's share of a batch included.
"""
import numpy as np
import pytest

from oracle import fixed_point as OFP
from test_gpu_spectral import (U32, contour, ctx, dev, fixed_point_bar, hf, host, inputs, make, relmax,  # noqa: F401
                               spectral_absrow, spectral_apply_bound, spectral_roundings, torch)

pytestmark = pytest.mark.gpu

# (nz, ny, nx): stages 8,8,2 / 8,4 / 7,5,3 / one stage / longest side 5^2 7 / planes near the limit
SHAPES = [(8, 32, 32), (7, 30, 42), (20, 63, 25), (9, 16, 49), (2, 24, 24), (105, 48, 27), (12, 128, 8), (6, 5, 175),
          (3, 96, 100), (128, 16, 20), (4, 140, 140)]


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("shape", SHAPES)
def test_products(ctx, shape, prec):  # noqa: F811
    o, g = make(ctx, shape, 21, 9.0)
    rng = np.random.default_rng(22)
    x = inputs(rng.standard_normal((2,) + shape) + 1j * rng.standard_normal((2,) + shape), prec)
    shift = 0.37 - 1.21j
    y = host(hf.apply(g, dev(x).to(torch.complex128 if prec == "f64" else torch.complex64), shift))
    unit = 1.0 if prec == "f32" else 2.0 ** -53 / U32
    for k in range(2):
        ref = o.apply(x[k], shift)
        bound = unit * spectral_apply_bound(x[k], float(o.lam.max()), o.kappa, o.damp, shift)
        assert np.abs(y[k] - ref).max() <= bound, (k, np.abs(y[k] - ref).max(), bound)


@pytest.mark.parametrize("prec,q,steps", [("f64", 8, 3), ("f64", 2, 3), ("f64", 1, 3), ("f32", 5, 3)])
def test_fixed_steps(ctx, prec, q, steps):  # noqa: F811
    o, g = make(ctx, (9, 21, 20), 25, 16.0)
    poles, cg = contour(o, g, 4, q)
    rng = np.random.default_rng(26)
    f = inputs(rng.standard_normal((2,) + o.shape) + 1j * rng.standard_normal((2,) + o.shape), prec)
    y, _ = hf.shifted_solve(g, cg, dev(f).to(torch.complex128 if prec == "f64" else torch.complex64), steps=steps)
    y = host(y)
    for j, p in enumerate(poles):
        for r in range(2):
            ref, _ = OFP.fixed_point_solve(o.apply, f[r], p.z, p.z0, p.delta, q, steps=steps)
            if prec == "f64":
                assert relmax(y[j, r], ref) <= 1e-11, (j, r)
            else:
                bar = fixed_point_bar(p, q, steps, o.rectangle(),
                                      spectral_absrow(float(o.lam.max()), o.kappa, o.rho2),
                                      np.linalg.norm(f[r]) / np.linalg.norm(ref), roundings=spectral_roundings(o.n))
                assert np.abs(y[j, r] - ref).max() <= bar * np.linalg.norm(ref), (j, r)


@pytest.mark.parametrize("q", [1, 2, 5])
def test_stopping_systems(ctx, q):  # noqa: F811
    """12 poles x 3 right-hand sides, one of them zero: systems leave the batch step by step."""
    o, g = make(ctx, (10, 18, 16), 27, 12.0)
    poles, cg = contour(o, g, 12, q)
    rng = np.random.default_rng(28)
    f = rng.standard_normal((3,) + o.shape) + 1j * rng.standard_normal((3,) + o.shape)
    f[1] = 0.0
    y, st = hf.shifted_solve(g, cg, dev(f), reduce=5.0, max_steps=60)
    y = host(y)
    for j, p in enumerate(poles):
        assert st[j, 1] == 0 and np.all(y[j, 1] == 0)
        for r in (0, 2):
            ref, hist = OFP.fixed_point_solve(o.apply, f[r], p.z, p.z0, p.delta, q, reduce=5.0, m_max=60)
            assert st[j, r] == len(hist) - 1, (j, r)
            assert relmax(y[j, r], ref) <= 1e-11, (j, r)
