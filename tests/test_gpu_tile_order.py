"""The pointwise passes of large grids on both sides of the rule that gives
them the stencil passes' tile order: tiles of 32 bytes of planes or more (8
planes in FP32, 4 in FP64).  The two forms add the same terms in another order.
"""
import pytest

from paper_2209_13768_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("method", ["bicgstab", "cg"])
@pytest.mark.parametrize("precision", ["f64", "f32"])
def test_both_sides_of_the_tile_order_rule(precision, method):
    """Five iterations on 64 x 64 x 1040 cells, 1040 tiles of 8 planes and more
    of fewer.  A dot product of n = 4.3e6 terms varies with its order by some
    sqrt(n) eps = 5e-13 at most; over five iterations, with what the
    well-conditioned system makes of it, x by 1e-11.  In FP32 a step length
    may also round to the next number, 1e-7: x by 1e-5."""
    import torch
    from paper_2209_13768_amd import wfa
    shape = (64, 64, 1040)
    u = (0.0, 0.0, 0.0) if method == "cg" else (1.0, -0.5, 0.25)
    h = inputs.grid_spacing(*shape)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)
    T0 = torch.rand(shape[::-1], generator=gen, device="cuda", dtype=torch.float64)
    xs = []
    for zc in ((7, 8) if precision == "f32" else (3, 4)):
        g = wfa.Grid(*shape, h=h, dt=0.5 * h * h, u=u, bc=inputs.MIXED_BC_KIND, precision=precision)
        g.set_option(wfa.OPT_ZCHUNK, zc)
        assert g.tiling()[3] >= 1024
        b = g.rhs(g.field(T0))
        x, info = g.solve(b, tol=1e-300, maxit=5, method=method, check=False)
        assert info.iterations == 5
        xs.append(x.double())
    rel = float((xs[0] - xs[1]).norm() / xs[1].norm())
    assert rel <= (1e-11 if precision == "f64" else 1e-5), rel
