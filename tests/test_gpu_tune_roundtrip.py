"""Reading an operator's launch shape and setting it again changes nothing (needs an MI355X)."""
import numpy as np
import pytest

from test_zz_no_alloc import ctx, dev, hf, setup, torch  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [32, 64])
@pytest.mark.parametrize("first", [None, (1, 4, 2, 0, 0, 1), (0, 4, 1, 5, 1, 2)])
def test_setting_the_shape_that_was_read_is_the_identity(ctx, prec, first):  # noqa: F811
    # bits, since the passes with several factors in registers round otherwise than single ones
    o, g, cg, poles, rng = setup(ctx, (20, 24, 70), 101, 8)
    if first is not None:
        g.set_tune(prec, *first)
    f = rng.standard_normal((2, 20, 24, 70)) + 1j * rng.standard_normal((2, 20, 24, 70))
    fd = dev(f).to(torch.complex64 if prec == 32 else torch.complex128)
    kw = dict(reduce=5.0, max_steps=60)
    y0, s0 = hf.shifted_solve(g, cg, fd, **kw)
    a0 = hf.apply(g, fd, 0.3 + 0.2j)
    shape = g.get_tune(prec)
    g.set_tune(prec, *shape)
    assert g.get_tune(prec) == shape
    y1, s1 = hf.shifted_solve(g, cg, fd, **kw)
    assert np.array_equal(s0, s1) and torch.equal(y0, y1)
    assert torch.equal(a0, hf.apply(g, fd, 0.3 + 0.2j))
    # from another shape back to the one read
    g.set_tune(prec, 1, 8, 3, 16, 0, 1)
    g.set_tune(prec, *shape)
    y2, s2 = hf.shifted_solve(g, cg, fd, **kw)
    assert np.array_equal(s0, s2) and torch.equal(y0, y2)
