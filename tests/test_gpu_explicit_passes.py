"""How wfa_explicit_step shares its steps out, and rows at the ends of the
fused pass's addressing: bitwise one pass per step.

The automatic choice fuses 1 to 4 steps by grid size and makes the number of
passes even where it can; a row longer than the buffer offsets' range (2^24 / 8
cells in FP32, 2^24 / 4 in FP64) goes by pointers.
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
    h = inputs.grid_spacing(*shape)
    g = wfa.Grid(*shape, h=h, dt=0.1 * h * h, u=(h, -2 * h, h), bc=inputs.MIXED_BC_KIND,
                 bc_value=(0.5, 0.25, 0, 0, 0, 0), precision=precision)
    g.set_option(wfa.OPT_EXPLICIT_FUSE, fuse)
    return g.explicit(T0.clone(), nsteps)


# 150^3 and 270^3 steps are fused by two in FP32 and by three in FP64
@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("shape", [(40, 30, 20), (150, 150, 150), (270, 250, 240)],
                         ids=["small", "150", "270"])
def test_automatic_fusing_is_bitwise_one_step_per_pass(wfa, precision, shape):
    import torch
    dtype = torch.float32 if precision == "f32" else torch.float64
    gen = torch.Generator(device="cuda")
    gen.manual_seed(11)
    T0 = torch.rand(shape[::-1], generator=gen, device="cuda", dtype=dtype)
    for nsteps in (0, 1, 2, 3, 4, 5, 7, 12):
        assert torch.equal(_run(wfa, shape, precision, nsteps, 0, T0),
                           _run(wfa, shape, precision, nsteps, 1, T0)), (precision, shape, nsteps)


@pytest.mark.parametrize("precision,rows", [("f32", 8), ("f64", 4)])
@pytest.mark.parametrize("over", [0, 1, 70])
def test_rows_at_the_range_of_buffer_offsets(wfa, precision, rows, over):
    import torch
    shape = ((1 << 24) // rows + over, 3, 2)
    dtype = torch.float32 if precision == "f32" else torch.float64
    gen = torch.Generator(device="cuda")
    gen.manual_seed(12)
    T0 = torch.rand(shape[::-1], generator=gen, device="cuda", dtype=dtype)
    for fuse in (2, 4):
        assert torch.equal(_run(wfa, shape, precision, 4, fuse, T0),
                           _run(wfa, shape, precision, 4, 1, T0)), (precision, over, fuse)
