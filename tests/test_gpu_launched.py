"""The launched kernels of the single-instance solves on lattices so small that
a call would otherwise take the persistent launch (DP_SMALL=0 keeps to them):
paired x updates on and off, mixed precision at every width, graph replay, the
solve without allocations and every stencil launch that the even-odd order
admits, on an even-odd lattice and on one with odd extents."""
import sys

import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2106_01275_amd as dp  # noqa: E402


def _say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def cuda(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.fixture(autouse=True)
def launched(monkeypatch):
    monkeypatch.setenv("DP_SMALL", "0")


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return dp.context(0)


DIMS = [(8, 6, 4, 4), (6, 4, 5, 4)]


def _system(dims, n, seed, links=True):
    rng = np.random.default_rng(seed)
    N = int(np.prod(dims))
    U = workloads.random_links(dims, 0.4, 6) if links else None
    return U, rng.standard_normal((n, N, 3)) + 1j * rng.standard_normal((n, N, 3))


@pytest.mark.parametrize("dims", DIMS)
@pytest.mark.parametrize("inner,graph", [("f32", 0), ("f32", 1), ("bf16", 0), ("bf16", 1)])
def test_paired_updates(ctx, monkeypatch, inner, graph, dims):
    """Both ways reach the oracle's solution (1e-8 at a true residual of 1e-10),
    a constant right-hand side of the free field (an eigenvector, whose beta is
    next to nothing) to 1e-9; and they do round differently, so the pairs ran."""
    _say("paired updates", inner, graph, dims)
    _, B = _system(dims, 40, 31)
    B[3] = 1.0 + 0.5j
    Xo, _, _ = oracle.cg_many(dims, 3, 0.1, None, B, tol=1e-13)
    op = ctx.operator(dims, 3, 0.1, None)
    got = []
    for pairs in ("1", "0"):
        monkeypatch.setenv("DP_XDEFER", pairs)
        (X,), (st,) = ctx.solve_batch([op], [cuda(B)], ctx.opts(tol=1e-10, inner=inner, rhs_block=32, use_graph=graph))
        got.append(X)
        X = X.cpu().numpy()
        assert st["nconverged"] == 40 and st["max_true_resid"] <= 1e-10 and st["reliable_updates"] >= 2
        assert np.abs(X - Xo).max() < 1e-8 * np.abs(Xo).max()
        assert np.abs(X[3] - Xo[3]).max() < 1e-9 * np.abs(Xo[3]).max()
    assert not torch.equal(got[0], got[1])


@pytest.mark.parametrize("dims", DIMS)
@pytest.mark.parametrize("inner", ["f32", "bf16"])
def test_paired_updates_at_every_stop(ctx, monkeypatch, inner, dims):
    """Stopped after k iterations (two a step in even-odd order), k = 1 .. 14, the
    iterate is the same with pairs and without, to the storage precision."""
    _say("every stop", inner, dims)
    U, B = _system(dims, 32, 41)
    op = ctx.operator(dims, 3, 0.1, cuda(U))
    for k in range(1, 15):
        xs = []
        for pairs in ("1", "0"):
            monkeypatch.setenv("DP_XDEFER", pairs)
            (X,), (st,) = ctx.solve_batch([op], [cuda(B)], ctx.opts(tol=1e-14, max_iter=k, inner=inner, rhs_block=32),
                                          check=False)
            assert st["max_iters"] == k if inner == "f32" else 0 < st["max_iters"] <= k
            xs.append(X)
        assert (xs[0] - xs[1]).abs().max() < (1e-5 if inner == "f32" else 5e-2) * xs[1].abs().max(), k


@pytest.mark.parametrize("dims", DIMS)
@pytest.mark.parametrize("inner", ["f64", "f32", "bf16"])
def test_every_width(ctx, inner, dims):
    """Blocks of 1 to 256 lanes, a part full last block: the oracle's solutions
    (FP64 1e-10 at 1e-12, mixed 1e-8 at 1e-10), and the solve without allocations,
    which runs the launches that the context chose before, to the bit."""
    _say("widths", inner, dims)
    U, B = _system(dims, 70, 12)
    op = ctx.operator(dims, 3, 0.1, cuda(U))
    Xo, _, _ = oracle.cg_many(dims, 3, 0.1, U, B, tol=1e-14)
    tol, bar = (1e-12, 1e-10) if inner == "f64" else (1e-10, 1e-8)
    for block in (1, 2, 4, 8, 16, 32, 64, 128, 256):
        n = 5 if block == 1 else 70
        o = ctx.opts(tol=tol, inner=inner, rhs_block=block)
        (X,), (st,) = ctx.solve_batch([op], [cuda(B[:n])], o)
        assert st["nconverged"] == n and st["max_true_resid"] <= tol * (10 if inner == "f64" else 1)
        assert np.abs(X.cpu().numpy() - Xo[:n]).max() < bar * np.abs(Xo).max(), block
        if block <= 32:
            Y, sy = ctx.solve_noalloc(op, cuda(B[:n]), o)
            assert sy["nconverged"] == n and sy["rhs_iters"] == st["rhs_iters"] and torch.equal(X, Y), block


@pytest.mark.parametrize("dims", DIMS)
@pytest.mark.parametrize("inner", ["f64", "f32", "bf16"])
def test_graph_replay_is_eager(ctx, inner, dims):
    """Groups of the predicted lengths replayed from graphs, several blocks and
    both solves of a gradient, with eager work between the replays: to the bit."""
    _say("graphs", inner, dims)
    U, B = _system(dims, 40, 3)
    col, m, _ = oracle.coloring(dims, 1, 2, oracle.NATURAL)
    op = ctx.operator(dims, 3, 0.1, cuda(U))
    ps = ctx.probe_spec(dims, 3, cuda(col), m, 5, 0, 2, "z2_complex", True)
    for block in (1, 32):
        eager, graph = (ctx.opts(tol=1e-10, inner=inner, rhs_block=block, use_graph=g) for g in (0, 1))
        b = cuda(B[:3] if block == 1 else B)

        def run(o):
            T, g, dU, dUb, st = ctx.trace_grad(op, ps, 1, o) if block > 1 else (0, 0, b, b, {"rhs_iters": 0})
            (X,), (s,) = ctx.solve_batch([op], [b], o)
            return [torch.tensor([T, g]), dU, dUb, X], (st["rhs_iters"] if block == 1 else 0, s["rhs_iters"])

        ref = run(eager)
        for _ in range(3):
            got = run(graph)
            assert all(torch.equal(x, y) for x, y in zip(got[0], ref[0])) and got[1] == ref[1], block
            again = run(eager)
            assert all(torch.equal(x, y) for x, y in zip(again[0], ref[0])), block


@pytest.mark.parametrize("dims", [(16, 4, 4, 4), (8, 6, 4, 10)])
@pytest.mark.parametrize("W,modes", [(1, (0, 5)), (8, (0,)), (16, (0, 1)), (32, (0, 1)), (64, (0, 1, 2)), (128, (0, 1, 2))])
def test_every_even_odd_stencil_launch(monkeypatch, dims, W, modes):
    """Each stencil mode that the even-odd order admits, on one workgroup, few and
    many, forced in turn: the oracle's solutions.  (The grouped modes 3, 4 and 6
    need the index order; forced here, the built-in choice runs.)"""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    n = min(W, 20)
    U, B = _system(dims, n, 7)
    Xo, _, _ = oracle.cg_many(dims, 3, 0.2, U, B, tol=1e-14)
    Ug, b = cuda(U), cuda(B)
    for mode in (*modes, 3):
        for grid in (0, 1, 8, 24, 1024):
            _say("stencil launch", dims, W, mode, grid)
            monkeypatch.setenv("DP_STENCIL", f"{mode},{grid}")
            c = dp.Context(0)
            op = c.operator(dims, 3, 0.2, Ug)
            for inner in ("f64", "f32", "bf16"):
                if mode == 5 and inner == "bf16":
                    continue
                tol, bar = (1e-12, 1e-10) if inner == "f64" else (1e-10, 1e-8)
                (X,), (st,) = c.solve_batch([op], [b], c.opts(tol=tol, inner=inner, rhs_block=W))
                assert st["nconverged"] == n
                assert np.abs(X.cpu().numpy() - Xo).max() < bar * np.abs(Xo).max(), (mode, grid, inner)
            c.close()
