"""Which solves iterate resident, and a resident launch that gives up.

A resident launch needs every workgroup on a CU.  Where one is missing the
others' bounded waits end, and the solve goes on from x with one launch per
pass.  With the workgroup missing from the first launch on, x is still the
initial guess, so the result is bit for bit that of one launch per pass.
"""
import pytest

from paper_2209_13768_amd import inputs

pytestmark = pytest.mark.gpu

METHODS = ["bicgstab", "bicgstab2", "cg", "cg1"]


@pytest.fixture(scope="module")
def wfa():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2209_13768_amd import wfa as w
    w.lib()
    return w


def _problem(shape, method, seed, cell=True):
    u = (0.0, 0.0, 0.0) if method.startswith("cg") else (1.0, -0.5, 0.25)
    return inputs.random_problem(seed, *shape, cell=cell, u=u, bc_kind=inputs.MIXED_BC_KIND)


def _same(a, b):
    import torch
    return bool(torch.equal(a.view(torch.uint8), b.view(torch.uint8)))


# 256 tiles are resident and 257 are not; tiles of up to 8 planes in FP64, 16 in FP32
SHAPES = [((1, 1, 1), {}, True, True), ((64, 8, 256), {"zc": 1}, True, True),
          ((64, 8, 257), {"zc": 1}, False, False), ((64, 64, 64), {}, True, True),
          ((128, 128, 128), {}, False, True), ((64, 40, 33), {"zc": 9}, False, True),
          ((64, 40, 33), {"zc": 17}, False, False), ((64, 40, 33), {"ry": 1}, False, False),
          ((160, 160, 160), {}, False, False)]


@pytest.mark.parametrize("shape,tiles,f64,f32", SHAPES,
                         ids=["x".join(map(str, s[0])) + "".join(s[1]) for s in SHAPES])
@pytest.mark.parametrize("method", METHODS)
@pytest.mark.parametrize("precision", ["f64", "f32", "f32_ir64"])
def test_which_solves_iterate_resident(wfa, precision, method, shape, tiles, f64, f32):
    if precision == "f32_ir64" and method == "cg":
        pytest.skip("no such refinement")
    for cell in (False, True):
        prob = _problem(shape, method, 31, cell)
        g = wfa.Grid.from_problem(prob, precision=precision)
        if "zc" in tiles:
            g.set_option(wfa.OPT_ZCHUNK, tiles["zc"])
        if "ry" in tiles:
            g.set_option(wfa.OPT_RY, tiles["ry"])
        b = g.rhs(g.field(prob.T0))
        for option, value, off in ((None, 0, False), (wfa.OPT_PROFILE, 1 << 20, True),
                                   (wfa.OPT_GRAPH, 1, True), (wfa.OPT_RECOMPUTE_T, 1, True)):
            if option is not None:
                g.set_option(option, value)
            g.solve(b, g.field(prob.T0), tol=1e-300, maxit=3, method=method, check=False)
            launches, gave_up = g.resident_stats(reset=True)
            expect = (f64 if precision == "f64" else f32) and not off
            assert (launches > 0) == expect and gave_up == 0, (option, launches)
            if option is not None:
                g.set_option(option, 0)


# one tile; planes of 2 to 16 a tile
@pytest.mark.parametrize("shape", [(5, 3, 2), (70, 45, 38), (57, 82, 90), (70, 45, 200)],
                         ids=["5", "70", "57", "200"])
@pytest.mark.parametrize("method", METHODS)
@pytest.mark.parametrize("precision", ["f64", "f32"])
def test_solve_goes_on_per_pass_when_a_launch_gives_up(wfa, precision, method, shape):
    prob = _problem(shape, method, 41)
    tol, maxit = (1e-10 if precision == "f64" else 1e-4), 2000
    g = wfa.Grid.from_problem(prob, precision=precision)
    b = g.rhs(g.field(prob.T0))
    xr, ir = g.solve(b, g.field(prob.T0), tol=tol, maxit=maxit, method=method)
    resident = precision == "f32" or g.tiling()[2] <= 8
    launches, gave_up = g.resident_stats(reset=True)
    assert ir.status == wfa.OK and (launches > 0) == resident and gave_up == 0
    if not resident or g.tiling()[3] == 1:   # a lone workgroup misses nobody
        return
    g.set_option(wfa.OPT_FORCE_GIVE_UP, 1)
    x, i = g.solve(b, g.field(prob.T0), tol=tol, maxit=maxit, method=method)
    assert g.resident_stats(reset=True) == (1, 1)
    assert _same(x, xr)
    for f in ("status", "iterations", "restarts", "rel_res_recursive", "rel_res_true"):
        assert getattr(i, f) == getattr(ir, f), f
    # the grid's next solves do not try again
    x, i = g.solve(b, g.field(prob.T0), tol=tol, maxit=maxit, method=method)
    assert g.resident_stats() == (0, 0) and _same(x, xr)


@pytest.mark.parametrize("option", ["OPT_PERSISTENT", "OPT_GRAPH"])
@pytest.mark.parametrize("method", METHODS)
def test_automatic_launch_forms_leave_small_grids_resident(wfa, method, option):
    for shape, resident in (((41, 30, 22), True), ((97, 88, 99), False)):
        prob = _problem(shape, method, 44)
        out = []
        for value in (0, -1):
            g = wfa.Grid.from_problem(prob, precision="f64")
            g.set_option(getattr(wfa, option), value)
            b = g.rhs(g.field(prob.T0))
            x, i = g.solve(b, g.field(prob.T0), tol=1e-300, maxit=20, method=method, check=False)
            assert (g.resident_stats()[0] > 0) == resident, (shape, value)
            out.append((x, i.iterations))
        assert out[0][1] == out[1][1] and _same(out[0][0], out[1][0]), shape


@pytest.mark.parametrize("method", METHODS)
def test_later_chunks_count_on_from_the_iterations_made(wfa, oracle_mod, method):
    """Chunks of four iterations, the workgroup missing from the second: the
    solve restarts from the iterates it has and meets its tolerance."""
    prob = _problem((41, 30, 22), method, 42)
    o = oracle_mod.Oracle(prob)
    g = wfa.Grid.from_problem(prob, precision="f64")
    g.set_option(wfa.OPT_CHECK_EVERY, 4)
    b = g.rhs(g.field(prob.T0))
    g.set_option(wfa.OPT_FORCE_GIVE_UP, 2)
    x, i = g.solve(b, g.field(prob.T0), tol=1e-10, maxit=2000, method=method)
    launches, gave_up = g.resident_stats()
    assert gave_up == 1 and launches == 2
    assert i.status == wfa.OK and i.iterations > 4
    # the recursive residual met 1e-10; the true one follows it to within 10x here
    assert o.true_relres(b.cpu().numpy(), x.cpu().numpy()) <= 1e-9
    assert i.rel_res_recursive <= 1e-10


def test_time_steps_and_refinement_after_a_give_up(wfa):
    for precision, method in (("f64", "bicgstab"), ("f32_ir64", "bicgstab2"), ("f32_ir64", "cg1")):
        prob = _problem((41, 30, 22), method, 43)
        out = []
        for n in (0, 1, 2):
            g = wfa.Grid.from_problem(prob, precision=precision)
            g.set_option(wfa.OPT_METHOD, {"bicgstab": wfa.METHOD_BICGSTAB,
                                          "bicgstab2": wfa.METHOD_BICGSTAB2,
                                          "cg1": wfa.METHOD_CG1}[method])
            g.set_option(wfa.OPT_FORCE_GIVE_UP, n)
            T = g.field(prob.T0)
            infos = g.timestep(T, 3, tol=1e-11, maxit=3000)
            assert g.resident_stats()[1] == (1 if n else 0)
            out.append((T, [(i.iterations, i.refinements) for i in infos]))
        for T, counts in out[1:]:
            assert counts == out[0][1], (precision, method)
            assert _same(T, out[0][0]), (precision, method)


def test_two_streams_whose_grids_do_not_fit_side_by_side(wfa):
    """160 workgroups of one per CU each, from two threads: each solve gives
    what it gives alone, in whichever form."""
    import threading
    import torch
    probs = [_problem((64, 64, 160), "cg1", 704 + 2 * q) for q in range(2)]

    def solve(prob, n):
        with torch.cuda.stream(torch.cuda.Stream()):
            g = wfa.Grid.from_problem(prob, precision="f64")
            b = g.rhs(g.field(prob.T0))
            return [g.solve(b, g.field(prob.T0), tol=1e-11, maxit=2000, method="cg1")[0].cpu()
                    for _ in range(n)]
    alone = [solve(p, 1)[0] for p in probs]
    got = [None, None]

    def work(q):
        got[q] = solve(probs[q], 8)
    ts = [threading.Thread(target=work, args=(q,)) for q in range(2)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    for q in range(2):
        assert all(torch.equal(x, alone[q]) for x in got[q])


def test_more_solves_at_once_than_fit_the_gpu(wfa):
    """Eight threads whose grids have 40 to 160 workgroups: solves that get no
    turn take one launch per pass, none waits in vain, and each gives what it
    gives alone."""
    import threading
    import torch
    shapes = [(64, 64, 160), (70, 45, 38), (40, 33, 21), (97, 61, 45)]
    probs = [_problem(shapes[q % 4], "cg1", 720 + q, cell=q % 2 == 0) for q in range(8)]

    def solve(prob, n):
        with torch.cuda.stream(torch.cuda.Stream()):
            g = wfa.Grid.from_problem(prob, precision="f64")
            b = g.rhs(g.field(prob.T0))
            xs = [g.solve(b, g.field(prob.T0), tol=1e-11, maxit=2000, method="cg1")[0].cpu()
                  for _ in range(n)]
            return xs, g.resident_stats()
    alone = [solve(p, 1)[0][0] for p in probs]
    got = [None] * 8

    def work(q):
        got[q] = solve(probs[q], 6)
    ts = [threading.Thread(target=work, args=(q,)) for q in range(8)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    for q in range(8):
        xs, (launches, gave_up) = got[q]
        assert all(torch.equal(x, alone[q]) for x in xs) and gave_up == 0, q
    assert sum(s[0] for _, s in got) > 0


def test_resident_solves_beside_persistent_launches_and_large_passes(wfa):
    """Other kernels that need or hold many CUs, from threads of their own: a
    persistent launch of as many workgroups, and the passes of a grid that
    fills the GPU.  Every solve gives what it gives alone."""
    import threading
    import torch
    small = _problem((64, 64, 160), "bicgstab", 731)
    large = _problem((200, 180, 160), "bicgstab2", 732)

    def solve(prob, method, persistent, n, maxit):
        with torch.cuda.stream(torch.cuda.Stream()):
            g = wfa.Grid.from_problem(prob, precision="f64")
            g.set_option(wfa.OPT_PERSISTENT, persistent)
            b = g.rhs(g.field(prob.T0))
            return [g.solve(b, g.field(prob.T0), tol=1e-300, maxit=maxit, method=method)[0].cpu()
                    for _ in range(n)]
    works = [(small, "bicgstab", 0, 12, 60), (small, "bicgstab", 1, 6, 60),
             (small, "bicgstab", 0, 12, 60), (large, "bicgstab2", 0, 4, 40)]
    alone = [solve(p, m, per, 1, k)[0] for p, m, per, _, k in works]
    got = [None] * len(works)

    def work(q):
        got[q] = solve(*works[q])
    ts = [threading.Thread(target=work, args=(q,)) for q in range(len(works))]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    for q in range(len(works)):
        assert got[q] is not None and all(_same(x, alone[q]) for x in got[q]), q
