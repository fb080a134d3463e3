"""Multi-factor passes with planes in registers against single factors (needs an MI355X).

An operator whose launch shape was never set, and the shapes with fuse 1 and kern 0 or 1, run
the fixed-point factors several per pass on 64-column tiles of waves stacked in y.  Every case
compares with the single-factor passes of the same operator (fuse 0) at grids where a tile, a
block or a z-chunk ends: x below, at and just past one 64-column tile and past two, y below a
block and with a ragged last one, one and few planes; degrees that split into every mixture of
two, three and four factors, one step (the two-output end) and several.

Bars: both sides evaluate the same product of q factors with the same coefficients.  In FP64
each is within 1e-12 of the oracle (the lockstep bar of the parity tests), so the two within
2e-12.  In FP32 each is within the product form's rounding bar of the oracle, so the two within
twice that.
"""
import numpy as np
import pytest

from oracle import fci as OF
from oracle import fixed_point as OFP
from oracle import operator as OO
from test_gpu_fullsize import ctx, dev, hf, host, round32, tol_of, torch  # noqa: F401

pytestmark = pytest.mark.gpu

SHAPES = [(5, 7, 63), (1, 9, 64), (9, 30, 65), (12, 49, 127), (3, 2, 130), (18, 61, 20)]


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("shape", SHAPES)
def test_register_passes_match_single_factors(ctx, shape, prec):  # noqa: F811
    rng = np.random.default_rng(sum(shape))
    c = rng.uniform(1.0, 3.0, size=shape)
    h = 1.0 / max(shape)
    o = OO.Operator(c, 0.3 / h, 2, 1.0, h=h)
    g = hf.Operator(ctx, dev(c), h, 0.3 / h, 2, 1.0)
    single = hf.Operator(ctx, dev(c), h, 0.3 / h, 2, 1.0)
    pr, dt = (64, torch.complex128) if prec == "f64" else (32, torch.complex64)
    single.set_tune(pr, 1, 4, 2, 0, 0)
    f = rng.standard_normal((2,) + shape) + 1j * rng.standard_normal((2,) + shape)
    f = round32(f) if prec == "f32" else f
    for q, steps in [(3, 2), (4, 3), (5, 1), (6, 2), (7, 3), (8, 2), (9, 1), (11, 2), (13, 2), (16, 2)]:
        poles = OF.pole_parameters(o, 4, 1.0, 0.5, q)
        kw = dict(z=[p.z for p in poles], sigma=[p.sigma for p in poles], delta=[p.delta for p in poles])
        cg, cs = hf.Contour(g, 4, 1.0, 0.5, q, **kw), hf.Contour(single, 4, 1.0, 0.5, q, **kw)
        ref, st = hf.shifted_solve(single, cs, dev(f).to(dt), steps=steps)
        ref = host(ref)
        for shp in (None, (0, 4, 1, 3, 1), (1, 8, 2, 0, 1)):
            if shp is None:
                gg, cc = g, cg
            else:
                gg = hf.Operator(ctx, dev(c), h, 0.3 / h, 2, 1.0)
                gg.set_tune(pr, *shp)
                cc = hf.Contour(gg, 4, 1.0, 0.5, q, **kw)
            y, st = hf.shifted_solve(gg, cc, dev(f).to(dt), steps=steps)
            y = host(y)
            assert np.all(st == steps)
            for j, p in enumerate(poles):
                scale = np.abs(ref[j]).max()
                if prec == "f64":
                    bar = 2e-12
                else:
                    exact, _ = OFP.fixed_point_solve(lambda v, sh: o.apply(v, sh), f[0], p.z, p.z0, p.delta, q, steps=steps)
                    bar = 2 * tol_of("f32", o, p, q, steps, f[0], exact)
                assert np.abs(y[j] - ref[j]).max() <= bar * scale, (shape, q, steps, shp, j)


def test_register_passes_stop_where_single_factors_do(ctx):  # noqa: F811
    # adaptive FP64: the same steps for every system (a zero right-hand side among them), with
    # the geometry of a pass changing as systems stop, and on a repeated call
    shape = (20, 40, 70)
    rng = np.random.default_rng(3)
    c = rng.uniform(1.0, 3.0, size=shape)
    h = 1.0 / 70
    g = hf.Operator(ctx, dev(c), h, 20.0, 3, 1.0)
    single = hf.Operator(ctx, dev(c), h, 20.0, 3, 1.0)
    single.set_tune(64, 1, 4, 2, 0, 0)
    f = rng.standard_normal((3,) + shape) + 1j * rng.standard_normal((3,) + shape)
    f[1] = 0.0
    out = []
    for op in (single, g, g):
        y, st = hf.shifted_solve(op, hf.Contour(op, 6, 1.0, 0.3, 8), dev(f), reduce=5.0, max_steps=80)
        out.append((host(y), st))
    assert np.array_equal(out[0][1], out[1][1]) and np.array_equal(out[1][1], out[2][1])
    assert len(set(out[0][1][:, 0].tolist())) > 1
    assert np.array_equal(out[1][0], out[2][0])
    assert np.abs(out[0][0] - out[1][0]).max() <= 1e-10 * np.abs(out[0][0]).max()


@pytest.mark.parametrize("q", [3, 8, 10])
@pytest.mark.parametrize("prec", [64, 32])
def test_batch_passes_match_single_operators(ctx, prec, q):  # noqa: F811
    # instances from one tile to several, a thin one, and one whose systems outlast the others
    # (the geometry changes with the work left): each against its own shifted solves, same
    # steps.  FP64 to 2e-12 of the largest value, FP32 to 1e-5: both sides are within the FP32
    # bar, at most 40 steps of q <= 10 products with errors of a few 6e-8 each
    shapes = [(3, 5, 70), (40, 33, 64), (1, 20, 21), (24, 60, 130)]
    dt = torch.complex128 if prec == 64 else torch.complex64
    ops, cons, fs = [], [], []
    rng = np.random.default_rng(q)
    for i, shape in enumerate(shapes):
        c = rng.uniform(1.0, 3.0, size=shape)
        h = 1.0 / max(shape)
        g = hf.Operator(ctx, dev(c), h, 0.3 / h, 2, 1.0)
        ops.append(g)
        cons.append(hf.Contour(g, 4 + 2 * (i % 2), 1.0, 0.25 if i == 1 else 0.6, q))
        f = rng.standard_normal(shape) + 1j * rng.standard_normal(shape)
        fs.append(dev(f).to(dt))
    ys, st = hf.shifted_solve_batch(ops, cons, fs, reduce=5.0, max_steps=40)
    assert max(int(s.max()) for s in st) > min(int(s.max()) for s in st)
    for g, c, f, y, s in zip(ops, cons, fs, ys, st):
        ref, rs = hf.shifted_solve(g, c, f[None], reduce=5.0, max_steps=40)
        if prec == 64:
            assert np.array_equal(s, rs[:, 0])
        same = s == rs[:, 0]  # (an FP32 residual can land on the other side of the threshold)
        assert same.sum() >= len(s) - 1
        a, b = host(y)[same], host(ref)[same, 0]
        assert np.abs(a - b).max() <= (2e-12 if prec == 64 else 1e-5) * np.abs(b).max()
