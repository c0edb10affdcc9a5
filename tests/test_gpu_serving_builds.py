"""The batched passes' builds for a batch of one kind of solves against the
build for any mix: a request served alone and beside a longer one of the other
kind of coefficients, which keeps the mixed build on, gives the same bits.
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


@pytest.mark.parametrize("precision", ["f64", "f32", "f32_ir64"])
@pytest.mark.parametrize("cell", [False, True], ids=["const", "cell"])
@pytest.mark.parametrize("u", [(0.0, 0.0, 0.0), (1.0, -0.5, 0.25)], ids=["diffusion", "convection"])
def test_one_kind_is_bitwise_the_mixed_build(wfa, precision, cell, u):
    import torch
    tol = {"f64": 1e-9, "f32": 1e-4, "f32_ir64": 1e-9}[precision]
    dtype = torch.float32 if precision == "f32" else torch.float64
    probs = [inputs.random_problem(71, 70, 17, 9, cell=cell, u=u, bc_kind=inputs.MIXED_BC_KIND,
                                   dt=1e-3),
             inputs.random_problem(72, 33, 8, 19, cell=cell, u=u, dt=1e-3)]
    other = inputs.random_problem(73, 64, 40, 40, cell=not cell, bc_kind=inputs.MIXED_BC_KIND,
                                  dt=1.0)
    got = []
    for mixed in (False, True):
        sv = wfa.Server(1 << 30, max_slots=4)
        reqs = probs + ([other] if mixed else [])
        fields = [torch.from_numpy(p.T0).to("cuda", dtype) for p in reqs]
        tickets = [sv.submit_problem(p, T, precision=wfa.PRECISIONS[precision], tol=tol, maxit=5000)
                   for p, T in zip(reqs, fields)]
        sv.drain()
        infos = [sv.poll(t) for t in tickets]
        sv.close()
        assert all(code == wfa.OK for code, _ in infos)
        if mixed:
            assert infos[2][1].iterations > max(i.iterations for _, i in infos[:2])
        got.append((fields[:2], [i.iterations for _, i in infos[:2]]))
    assert got[0][1] == got[1][1]
    for a, b in zip(got[0][0], got[1][0]):
        assert torch.equal(a, b)
