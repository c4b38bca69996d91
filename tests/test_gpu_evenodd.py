"""Solves on the even-odd reduced system (every extent even) against the
oracle's FP64 CG on the whole operator: extents of 2 (both hops of a
direction reach the same site), slabs of one and several x0-slices, part
tiles, every kind of block width, right-hand sides supported on one parity
only, and a zero one; with the launched kernels (DP_SMALL=0) and, for these
small lattices, one persistent launch per block.  Solutions to the bars of the other solve tests: 1e-10
(FP64 to 1e-12), 1e-8 (mixed to 1e-10)."""
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


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return dp.context(0)


def _rhs(dims, nc, n, seed):
    rng = np.random.default_rng(seed)
    N = int(np.prod(dims))
    B = rng.standard_normal((n, N, nc)) + 1j * rng.standard_normal((n, N, nc))
    parity = np.indices(dims).sum(0).ravel() % 2
    B[0][parity == 0] = 0  # odd sites only
    if n > 1:
        B[1][parity == 1] = 0
    if n > 2:
        B[2] = 0
    return B


@pytest.mark.parametrize("dims,nc,links,n,block", [((2, 2, 2, 2), 3, True, 3, 1), ((2, 2, 2, 2), 1, False, 1, 0),
                                                   ((4, 2, 6, 2), 3, True, 21, 8), ((6, 4, 2, 10), 3, True, 35, 16),
                                                   ((8, 2, 4, 6), 1, True, 33, 32), ((16, 2, 2, 4), 3, True, 40, 32),
                                                   ((8, 4, 4, 2), 3, False, 70, 64), ((4, 4, 2, 4), 3, True, 130, 128)])
@pytest.mark.parametrize("inner", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("small", ["0", "1"])
def test_reduced_solve_matches_oracle(ctx, monkeypatch, small, inner, dims, nc, links, n, block):
    _say("even-odd solve", inner, dims, nc, links, n, block, "small", small)
    monkeypatch.setenv("DP_SMALL", small)
    U = workloads.random_links(dims, 0.4, 5, nc) if links else None
    B = _rhs(dims, nc, n, 3)
    op = ctx.operator(dims, nc, 0.2, None if U is None else cuda(U))
    tol = 1e-12 if inner == "f64" else 1e-10
    o = ctx.opts(tol=tol, inner=inner, rhs_block=block)
    (X,), (st,) = ctx.solve_batch([op], [cuda(B)], o)
    Xo, _, _ = oracle.cg_many(dims, nc, 0.2, U, B, tol=1e-14)
    assert st["nconverged"] == n and st["max_true_resid"] <= tol * (10 if inner == "f64" else 1)
    err = np.abs(X.cpu().numpy() - Xo).max() / np.abs(Xo).max()
    assert err < (1e-10 if inner == "f64" else 1e-8), err


@pytest.mark.parametrize("inner", ["f64", "bf16"])
def test_batch_of_even_and_odd_extents(ctx, inner):
    """One call whose instances do and do not take the reduced system, in
    turn: dense right-hand sides against the oracle, each instance's result
    in its own place; a batch of one zero right-hand side each gives zeros."""
    _say("batch, even and odd extents", inner)
    shapes = [(4, 4, 4, 3), (4, 2, 6, 4), (5, 4, 2, 3), (8, 4, 2, 2), (2, 2, 4, 2)]
    counts = [5, 40, 17, 33, 1]
    Us = [workloads.random_links(d, 0.4, 40 + i) for i, d in enumerate(shapes)]
    Bs = [_rhs(d, 3, n, i) for i, (d, n) in enumerate(zip(shapes, counts))]
    ops = [ctx.operator(d, 3, 0.1 + 0.1 * i, cuda(Us[i])) for i, d in enumerate(shapes)]
    tol = 1e-12 if inner == "f64" else 1e-10
    o = ctx.opts(tol=tol, inner=inner, rhs_block=16)
    Xs, sts = ctx.solve_batch(ops, [cuda(b) for b in Bs], o)
    for i, d in enumerate(shapes):
        Xo, _, _ = oracle.cg_many(d, 3, 0.1 + 0.1 * i, Us[i], Bs[i], tol=1e-14)
        assert sts[i]["nconverged"] == sts[i]["nrhs"] == counts[i], i
        err = np.abs(Xs[i].cpu().numpy() - Xo).max() / np.abs(Xo).max()
        assert err < (1e-10 if inner == "f64" else 1e-8), (i, err)
    Zs, sts = ctx.solve_batch(ops, [torch.zeros_like(cuda(b[:1])) for b in Bs], o)
    assert all(torch.all(z == 0) for z in Zs) and all(s["nconverged"] == 1 for s in sts)


@pytest.mark.parametrize("small", ["0", "1"])
def test_reduced_failure_statuses(ctx, monkeypatch, small):
    """An indefinite operator breaks down and an iteration limit is kept, as
    on the whole operator."""
    monkeypatch.setenv("DP_SMALL", small)
    dims = (4, 4, 2, 4)
    B = cuda(_rhs(dims, 3, 5, 9)[3:])
    U = cuda(workloads.random_links(dims, 0.2, 2))
    for inner in ("f64", "f32", "bf16"):
        with pytest.raises(dp.DPError) as e:
            ctx.solve_batch([ctx.operator(dims, 3, -4.0, U)], [B], ctx.opts(tol=1e-10, inner=inner, max_iter=200))
        assert e.value.status == (dp.EBREAKDOWN if inner == "f64" else dp.ENOCONV), inner
        for k in (1, 2, 3):
            _, (st,) = ctx.solve_batch([ctx.operator(dims, 3, 0.1, U)], [B],
                                       ctx.opts(tol=1e-13, inner=inner, max_iter=k), check=False)
            assert st["nconverged"] == 0 and st["max_iters"] <= k
