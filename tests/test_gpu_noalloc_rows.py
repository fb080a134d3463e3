"""hfci_shifted_solve_noalloc with several tiles of the register passes (needs an MI355X).

The grids of tests/test_zz_no_alloc.py fit in one 64-column tile.  Here the tiles overlap in x
(and y), so that a residual pass has more blocks than the single-factor kernels have tiles, on
operators whose launch shape was never set (several factors per pass) and with z-chunks given.
The entry point runs the shifted solve's launches on other buffers: iterates and step counts
must be equal bit for bit, adaptive and at fixed counts, with many systems and with few left.
"""
import numpy as np
import pytest

from test_zz_no_alloc import ctx, dev, hf, setup, torch  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [32, 64])
@pytest.mark.parametrize("shape,tune", [((8, 8, 128), None), ((8, 8, 65), None), ((8, 8, 256), None),
                                        ((5, 9, 130), None), ((24, 40, 128), (1, 8, 2, 16, 1, 1)),
                                        ((48, 24, 66), (0, 4, 1, 7, 1, 2))])
def test_noalloc_equals_shifted_solve_across_tiles(ctx, shape, tune, prec):  # noqa: F811
    dt = torch.complex64 if prec == 32 else torch.complex128
    for q in (3, 8):
        o, g, cg, poles, rng = setup(ctx, shape, 90 + q, q, J=4)
        if tune is not None:
            g.set_tune(prec, *tune)
        f = rng.standard_normal((2,) + shape) + 1j * rng.standard_normal((2,) + shape)
        f[1] *= 1e-3
        fd = dev(f).to(dt)
        for kw in (dict(reduce=5.0, max_steps=60), dict(steps=3)):
            y_ref, st_ref = hf.shifted_solve(g, cg, fd, **kw)
            y = torch.full_like(y_ref, float("nan"))
            st = hf.shifted_solve_noalloc(g, cg, fd, y, **kw)
            assert np.array_equal(st, st_ref), (q, kw)
            assert torch.equal(y, y_ref), (q, kw)


def test_noalloc_with_many_systems_on_a_thin_grid(ctx):  # noqa: F811
    # 12 poles x 4 sources on 128 x 8 x 8 points: 48 systems of three blocks each
    o, g, cg, poles, rng = setup(ctx, (8, 8, 128), 97, 8, J=12)
    f = rng.standard_normal((4, 8, 8, 128)) + 1j * rng.standard_normal((4, 8, 8, 128))
    fd = dev(f).to(torch.complex64)
    y_ref, st_ref = hf.shifted_solve(g, cg, fd, reduce=5.0, max_steps=60)
    y = torch.full_like(y_ref, float("nan"))
    st = hf.shifted_solve_noalloc(g, cg, fd, y, reduce=5.0, max_steps=60)
    assert np.array_equal(st, st_ref) and torch.equal(y, y_ref)
