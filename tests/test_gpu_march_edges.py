"""The stencil passes at the edges of their tiles (64 x 8 cells), where the
engine that tests whole waves for the grid's faces changes between its
branches: against the same passes with four rows per wave, which test by
lanes.

The operator's and an explicit step's values are formed by the same operations
in both and agree bitwise.  A solve's sums are added in another order, some
1e-16 of their size, and two iterations carry that into x at most a few
hundredfold: 1e-12 in FP64; in FP32 a scalar may round the other way, 1e-7, so
2e-5.
"""
import pytest

from paper_2209_13768_amd import inputs

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1, 1), (63, 7, 2), (64, 8, 3), (65, 9, 1), (128, 16, 5), (129, 17, 4), (192, 25, 3),
          (193, 2, 19)]
PHYSICS = {
    "const_diffusion": dict(cell=False, u=(0.0, 0.0, 0.0), bc_kind=inputs.MIXED_BC_KIND),
    "const_upwind": dict(cell=False, u=(0.5, -1.0, 0.25), bc_kind=(inputs.DIRICHLET,) * 6),
    "cell_diffusion": dict(cell=True, u=(0.0, 0.0, 0.0), bc_kind=(inputs.DIRICHLET,) * 6),
    "cell_upwind": dict(cell=True, u=(1.0, 0.5, -0.25), bc_kind=inputs.MIXED_BC_KIND),
}


@pytest.fixture(scope="module")
def wfa():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2209_13768_amd import wfa as w
    w.lib()
    return w


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("name", sorted(PHYSICS))
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_two_rows_per_wave_match_four(wfa, precision, name, shape):
    import torch
    prob = inputs.random_problem(31, *shape, dt=1e-3, **PHYSICS[name])
    tol = 1e-12 if precision == "f64" else 2e-5
    res = []
    for ry in (2, 4):
        g = wfa.Grid(*shape, h=prob.h, dt=prob.dt, alpha=prob.alpha,
                     kappa=None if prob.kappa is None else torch.as_tensor(prob.kappa).cuda(),
                     u=prob.u, bc=prob.bc_kind, bc_value=prob.bc_value, precision=precision)
        g.set_option(wfa.OPT_RY, ry)
        g.set_option(wfa.OPT_EXPLICIT_FUSE, 1)
        g.set_option(wfa.OPT_PROFILE, 1)   # a launch per pass
        T0 = torch.as_tensor(prob.T0).cuda().to(g.dtype)
        exact = [g.apply(T0, g.field()).clone(), g.explicit(T0.clone(), 2).clone()]
        b = g.rhs(T0)
        solved = []
        for jacobi in (0, 1):
            g.set_option(wfa.OPT_JACOBI, jacobi)
            for method in ("bicgstab", "bicgstab2") + (() if any(prob.u) or jacobi else ("cg", "cg1")):
                x = g.field()
                x.copy_(T0)
                g.solve(b, x, tol=1e-300, maxit=2, method=method, check=False)
                solved.append(((method, jacobi), x.clone()))
        res.append((exact, solved))
    for a, c in zip(res[0][0], res[1][0]):
        assert torch.equal(a, c)
    for (what, a), (_, c) in zip(res[0][1], res[1][1]):
        assert torch.isfinite(a).all(), what
        err = float((a - c).double().norm() / c.double().norm())
        assert err <= tol, (what, err)
