"""The steps per pass that WFA_OPT_EXPLICIT_FUSE sets are the ones that run,
at any size: counted by launches, and bitwise one pass per step.
"""
import pytest

from paper_2209_13768_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def wfa():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2209_13768_amd import wfa as w
    w.lib()
    return w


def _run(wfa, shape, precision, nsteps, fuse, T0):
    """The field after nsteps, and the launches of fused and single steps."""
    h = inputs.grid_spacing(*shape)
    g = wfa.Grid(*shape, h=h, dt=0.1 * h * h, u=(h, -2 * h, h), bc=inputs.MIXED_BC_KIND,
                 bc_value=(0.5, 0.25, 0, 0, 0, 0), precision=precision)
    g.set_option(wfa.OPT_EXPLICIT_FUSE, fuse)
    g.set_option(wfa.OPT_PROFILE, 1)
    T = g.explicit(T0.clone(), nsteps)
    return T, g.kernel_stats(wfa.K_EXPLICIT_FUSED)[0], g.kernel_stats(wfa.K_EXPLICIT)[0]


def _field(shape, precision):
    import torch
    gen = torch.Generator(device="cuda")
    gen.manual_seed(13)
    return torch.rand(shape[::-1], generator=gen, device="cuda",
                      dtype=torch.float32 if precision == "f32" else torch.float64)


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("fuse", [1, 2, 3, 4])
def test_steps_per_pass_are_those_set(wfa, precision, fuse):
    import torch
    shape = (70, 45, 38)
    T0 = _field(shape, precision)
    for nsteps in (0, 1, 2, 3, 4, 6, 7, 9, 12):
        T, fused, single = _run(wfa, shape, precision, nsteps, fuse, T0)
        expect = (nsteps // fuse, nsteps % fuse) if fuse > 1 else (0, nsteps)
        assert (fused, single) == expect, (nsteps, fused, single)
        assert torch.equal(T, _run(wfa, shape, precision, nsteps, 1, T0)[0]), nsteps


# a row at, one past and 70 past the range of the buffer offsets (2^24 / 8
# cells in FP32, 2^24 / 4 in FP64), where rows go by pointers
@pytest.mark.parametrize("precision,rows", [("f32", 8), ("f64", 4)])
@pytest.mark.parametrize("over", [0, 1, 70])
@pytest.mark.parametrize("fuse", [2, 3, 4])
def test_every_depth_at_the_range_of_buffer_offsets(wfa, precision, rows, over, fuse):
    import torch
    shape = ((1 << 24) // rows + over, 3, 2)
    T0 = _field(shape, precision)
    T, fused, single = _run(wfa, shape, precision, 2 * fuse, fuse, T0)
    assert (fused, single) == (2, 0)
    assert torch.equal(T, _run(wfa, shape, precision, 2 * fuse, 1, T0)[0])


@pytest.mark.parametrize("fuse", [2, 3, 4])
@pytest.mark.parametrize("kind", ["zero-flux", "dirichlet"])
def test_a_ghost_value_past_fp32_stays_at_its_face(wfa, kind, fuse):
    """1e300 is infinite in FP32: ignored on a zero-flux face, and on a
    Dirichlet face what the cells next to it see, not the rest of their rows
    and planes."""
    import torch
    shape = (70, 45, 38)
    h = inputs.grid_spacing(*shape)
    T0 = _field(shape, "f32")
    for face in range(6):
        out = []
        for n in (1, fuse):
            bc = [wfa.BC_DIRICHLET] * 6
            if kind == "zero-flux":
                bc[face] = wfa.BC_ZEROFLUX
            g = wfa.Grid(*shape, h=h, dt=0.1 * h * h, bc=bc, precision="f32",
                         bc_value=[1e300 if f == face else 0.5 for f in range(6)])
            g.set_option(wfa.OPT_EXPLICIT_FUSE, n)
            out.append(g.explicit(T0.clone(), 2 * fuse))
        a, b = out
        finite = torch.isfinite(a)
        assert torch.equal(finite, torch.isfinite(b)), face
        assert torch.equal(a[finite], b[finite]), face
        # a step carries the face's infinity one cell further
        assert int((~finite).sum()) == (0 if kind == "zero-flux" else
                                        2 * fuse * (T0.numel() // shape[face // 2])), face
