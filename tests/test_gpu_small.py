"""Small problems, whose solve is one persistent launch per block, against the
oracle: one, two and four right-hand sides per group of workgroups, one and
several groups, more right-hand sides than run side by side, a last workgroup
with part of its sites, even-odd and index order, all three sources of the
right-hand sides (vectors, probes, deflated probes) and the mixed-precision
stopping rule.  FP64 throughout, so the FP64 bars hold for every precision
asked for (1e-10 at a residual of 1e-12; 1e-8 at 1e-10)."""
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


# (even-odd: 64 sites of a half per workgroup; index order: 64 sites)
@pytest.mark.parametrize("dims,nc,links,n,block", [((2, 2, 2, 2), 1, True, 2, 0),    # 8 sites, one workgroup
                                                   ((6, 4, 2, 6), 3, True, 1, 0),    # 144 sites: three, the last part full
                                                   ((8, 8, 8, 8), 3, True, 9, 0),    # 32 workgroups a group: two lanes each
                                                   ((8, 8, 8, 8), 3, True, 20, 32),  # four lanes each
                                                   ((4, 4, 4, 4), 3, False, 40, 8),  # several blocks
                                                   ((12, 8, 8, 8), 3, True, 15, 16),  # 48 a group: five groups
                                                   ((3, 5, 4, 3), 3, True, 7, 0), ((5, 3, 3, 5), 1, False, 33, 64),
                                                   ((9, 8, 7, 6), 3, True, 5, 0), ((1, 3, 2, 5), 3, True, 3, 4)])
@pytest.mark.parametrize("inner", ["f64", "f32"])
def test_small_solve_matches_oracle(ctx, inner, dims, nc, links, n, block):
    _say("small solve", inner, dims, nc, links, n, block)
    N = int(np.prod(dims))
    rng = np.random.default_rng(8)
    U = workloads.random_links(dims, 0.4, 6, nc) if links else None
    B = rng.standard_normal((n, N, nc)) + 1j * rng.standard_normal((n, N, nc))
    op = ctx.operator(dims, nc, 0.2, None if U is None else cuda(U))
    tol = 1e-12 if inner == "f64" else 1e-10
    o = ctx.opts(tol=tol, inner=inner, rhs_block=block)
    (X,), (st,) = ctx.solve_batch([op], [cuda(B)], o)
    Xo, _, _ = oracle.cg_many(dims, nc, 0.2, U, B, tol=1e-14)
    assert st["nconverged"] == n and st["max_true_resid"] <= tol * (10 if inner == "f64" else 1)
    assert (st["reliable_updates"] >= 1) == (inner == "f32")
    err = np.abs(X.cpu().numpy() - Xo).max() / np.abs(Xo).max()
    assert err < (1e-10 if inner == "f64" else 1e-8), err
    (X2,), (st2,) = ctx.solve_batch([op], [cuda(B)], o)
    assert torch.equal(X, X2) and st2["rhs_iters"] == st["rhs_iters"]


def test_small_sources_match_launched_kernels(ctx, monkeypatch):
    """Probes, shifted probes (the adjoint) and deflated probes: the same
    estimates and gradients as with the launched kernels."""
    _say("small sources")
    for dims in ((4, 4, 4, 4), (4, 3, 4, 5)):
        U = workloads.random_links(dims, 0.4, 3)
        col, m, _ = oracle.coloring(dims, 1, 2, oracle.NATURAL)
        op = ctx.operator(dims, 3, 0.3, cuda(U))
        ps = ctx.probe_spec(dims, 3, cuda(col), m, 5, 0, 1, "z2_complex", True)
        o = ctx.opts(tol=1e-12)
        d = ctx.deflation(op, 6, tol=1e-8, seed=2)
        got = {}
        for small in ("1", "0"):
            monkeypatch.setenv("DP_SMALL", small)
            T, g, dU, dUb, st = ctx.trace_grad(op, ps, 1, o)
            t = ctx.trace_deflated(op, d, 1, ps, o)
            got[small] = (ctx.trace_estimate([op], [ps], [1], o)[0]["tj"], st["tj"], dU.cpu().numpy(), dUb.cpu().numpy(),
                          t["tj"], np.array([T, g, t["T"]]))
        for a, b in zip(got["1"], got["0"]):
            assert np.abs(a - b).max() < 1e-10 * np.abs(b).max(), dims


def test_small_solve_gives_way(ctx, monkeypatch):
    """A persistent launch whose waits run out at once (no polls allowed) ends,
    and the call is solved by the launched kernels, with their very result."""
    _say("small solve gives way")
    dims, n = (6, 4, 4, 4), 5
    rng = np.random.default_rng(4)
    U = workloads.random_links(dims, 0.4, 3)
    B = cuda(rng.standard_normal((n, 384, 3)) + 1j * rng.standard_normal((n, 384, 3)))
    op = ctx.operator(dims, 3, 0.2, cuda(U))
    for inner in ("f64", "f32"):
        o = ctx.opts(tol=1e-11, inner=inner, rhs_block=8)
        monkeypatch.setenv("DP_SMALL", "0")
        (X0,), _ = ctx.solve_batch([op], [B], o)
        (N0,) = ctx.solve_noalloc(op, B, o)[:1]
        monkeypatch.setenv("DP_SMALL", "1")
        (X1,), _ = ctx.solve_batch([op], [B], o)
        monkeypatch.setenv("DP_SMALL_POLLS", "0")
        (X2,), st = ctx.solve_batch([op], [B], o)
        (N2,) = ctx.solve_noalloc(op, B, o)[:1]
        monkeypatch.delenv("DP_SMALL_POLLS")
        assert torch.equal(X2, X0) and torch.equal(N2, N0) and st[0]["nconverged"] == n
        assert (X1 - X0).abs().max() < 1e-9 * X0.abs().max()
        (X3,), _ = ctx.solve_batch([op], [B], o)
        assert torch.equal(X3, X1)
