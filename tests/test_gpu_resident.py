"""Resident iterations of small grids against one launch per pass, bit for bit.

Grids whose tiles fit on the chip iterate in one cooperative launch per chunk
with the vectors in registers; with per-launch timing on, the same solve runs
one launch per pass.  Both hold the same tiles, reduction orders and
finalizers, so every iterate, report and stored vector must be equal.  The
shapes are the edges of the rule and of the tiles: one cell, rows and planes
left over in x, y and z, one tile, several tiles in x, tiles of 1 to 16
planes (FP64 iterates resident up to 8), and the most tiles.
"""
import pytest

from paper_2209_13768_amd import inputs

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1, 1), (5, 3, 2), (64, 8, 4), (33, 17, 5), (70, 45, 38), (97, 61, 45), (64, 64, 64),
          (130, 9, 7), (3, 3, 300), (48, 48, 48), (200, 120, 9), (57, 82, 90), (70, 45, 200),
          (128, 128, 128)]
METHODS = ["bicgstab", "bicgstab2", "bicgstab2_hashed", "cg", "cg1"]


@pytest.fixture(scope="module")
def wfa():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2209_13768_amd import wfa as w
    w.lib()
    return w


def _grid(wfa, prob, precision, method, per_pass, jacobi=0):
    g = wfa.Grid.from_problem(prob, precision=wfa.PRECISIONS[precision])
    g.set_option(wfa.OPT_SHADOW, 1 if method == "bicgstab2_hashed" else 0)
    g.set_option(wfa.OPT_JACOBI, jacobi)
    if per_pass:
        g.set_option(wfa.OPT_PROFILE, 1 << 20)
    return g


def _problem(shape, method, seed):
    u = (0.0, 0.0, 0.0) if method.startswith("cg") else (1.0, -0.5, 0.25)
    return inputs.random_problem(seed, *shape, cell=seed % 2 == 0, u=u,
                                 bc_kind=inputs.MIXED_BC_KIND)


def _same(a, b):
    import torch
    return bool(torch.equal(a.view(torch.uint8), b.view(torch.uint8)))


@pytest.mark.parametrize("shape", SHAPES, ids=["x".join(map(str, s)) for s in SHAPES])
@pytest.mark.parametrize("method", METHODS)
@pytest.mark.parametrize("precision", ["f64", "f32"])
def test_resident_is_bitwise_one_launch_per_pass(wfa, precision, method, shape):
    name = method.split("_")[0]
    for seed in (700, 701):
        prob = _problem(shape, method, seed)
        tols = ((1e-300, 5, 0), (1e-300, 7, 3), (1e-4 if precision == "f32" else 1e-9, 3000, 0))
        for tol, maxit, every in tols[:2] if prob.cells > 10 ** 6 else tols:
            out = []
            for per_pass in (False, True):
                g = _grid(wfa, prob, precision, method, per_pass)
                g.set_option(wfa.OPT_CHECK_EVERY, every)
                b = g.rhs(g.field(prob.T0))
                x, info = g.solve(b, g.field(prob.T0), tol=tol, maxit=maxit, method=name, check=False)
                # (v is no vector of classic CG's)
                vecs = ([g.vector(q).clone() for q in (wfa.VEC_V0, wfa.VEC_V1)]
                        if maxit < 10 and name != "cg" else [])
                out.append((x, info, vecs))
            (xa, ia, va), (xb, ib, vb) = out
            what = (precision, method, shape, seed, tol, ia, ib)
            assert _same(xa, xb), what
            for f in ("status", "iterations", "restarts", "rel_res_recursive", "rel_res_true"):
                p, q = getattr(ia, f), getattr(ib, f)
                assert p == q or (p != p and q != q), what
            if ia.iterations == maxit:
                assert all(_same(p, q) for p, q in zip(va, vb)), what


def test_resident_jacobi_restart_refinement_and_reuse(wfa):
    prob = _problem((41, 30, 22), "bicgstab2", 702)
    out = []
    for per_pass in (False, True):
        xs = []
        g = _grid(wfa, prob, "f64", "bicgstab2_hashed", per_pass, jacobi=1)
        b = g.rhs(g.field(prob.T0))
        for k in range(3):          # the same grid again: slots, hints and buffers reused
            x, info = g.solve(b, g.field(prob.T0) * (k + 1), tol=1e-10, maxit=2000, method="bicgstab2")
            xs.append((x, info))
        g.set_option(wfa.OPT_FORCE_BREAKDOWN, 4)
        xs.append(g.solve(b, g.field(prob.T0), tol=1e-10, maxit=2000, method="bicgstab2"))
        assert xs[-1][1].restarts == 1
        for method in ("bicgstab2", "cg1"):
            sym = _problem((41, 30, 22), method, 702)
            g = _grid(wfa, sym, "f32_ir64", method, per_pass)
            g.set_option(wfa.OPT_FORCE_DIVERGE, 6)
            b2 = g.rhs(g.field(sym.T0))
            xs.append(g.solve(b2, g.field(sym.T0), tol=1e-12, maxit=5000, method=method))
        out.append(xs)
    for (xa, ia), (xb, ib) in zip(*out):
        assert ia.status == wfa.OK and (ia.iterations, ia.refinements) == (ib.iterations, ib.refinements)
        assert _same(xa, xb), (ia, ib)


def test_resident_solves_on_two_streams_and_threads(wfa):
    """Two grids iterate from two threads on streams of their own; each gives
    what it gives alone."""
    import threading
    import torch
    probs = [_problem((40, 33, 21 + 4 * q), "cg1", 704 + q) for q in range(2)]

    def solve(prob, n):
        s = torch.cuda.Stream()
        with torch.cuda.stream(s):
            g = _grid(wfa, prob, "f64", "cg1", False)
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
