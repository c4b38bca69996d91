"""The iteration limit and the iteration counts of a solve: the largest limit
there is does not end a solve early, and a step of the even-odd reduced system
counts as two iterations, so that a solve reports about as many as CG on the
whole operator takes (the oracle's).  The reduced system's Krylov space after n
steps holds that of n steps more on A, so CG on A needs at most two iterations
more than reported; it may need fewer where its last step falls between two of
the reduced system's or its residual (on all sites) dips earlier: bar one step,
and a quarter for the mixed-precision solves' extra steps after their updates."""
import sys

import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2106_01275_amd as dp  # noqa: E402


def cuda(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return dp.context(0)


@pytest.mark.parametrize("dims", [(4, 4, 6, 4), (4, 3, 5, 4)])
@pytest.mark.parametrize("inner", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("small", ["0", "1"])
def test_largest_limit_and_counts(ctx, monkeypatch, small, inner, dims):
    print("iteration limit", small, inner, dims, flush=True)
    sys.stdout.flush()
    monkeypatch.setenv("DP_SMALL", small)
    rng = np.random.default_rng(5)
    n, N = 6, int(np.prod(dims))
    U = workloads.random_links(dims, 0.4, 3)
    B = rng.standard_normal((n, N, 3)) + 1j * rng.standard_normal((n, N, 3))
    op = ctx.operator(dims, 3, 0.2, cuda(U))
    tol = 1e-12 if inner == "f64" else 1e-10
    Xo, _, _ = oracle.cg_many(dims, 3, 0.2, U, B, tol=1e-14)
    _, its, _ = oracle.cg_many(dims, 3, 0.2, U, B, tol=tol)
    o = ctx.opts(tol=tol, inner=inner, rhs_block=8, max_iter=2 ** 31 - 1)
    got = [(x, st) for xs, sts in [ctx.solve_batch([op], [cuda(B)], o), ctx.solve_batch([op] * 2, [cuda(B)] * 2, o)]
           for x, st in zip(xs, sts)] + [ctx.solve_noalloc(op, cuda(B), o)]
    for k, (x, st) in enumerate(got):
        assert st["nconverged"] == n, k
        err = np.abs(x.cpu().numpy() - Xo).max() / np.abs(Xo).max()
        assert err < (1e-10 if inner == "f64" else 1e-8), (k, err)
        if inner != "bf16":
            slack = 2 if inner == "f64" else 2 + its.max() // 4
            assert its.max() - 2 <= st["max_iters"] <= its.max() + slack, (k, st["max_iters"], its)
        if all(d % 2 == 0 for d in dims):
            assert st["rhs_iters"] % 2 == 0, k
