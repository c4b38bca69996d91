"""Persistent solves of blocks that take several rounds of lanes, whose last
round is part full, or whose width is mostly padding, and calls of many narrow
blocks: the choice and the shape of a launch go by the right-hand sides of a
block.  FP64 bars (1e-10 of the largest value at a residual of 1e-12).  The
launched kernels round differently, so equal bits would tell that the
persistent launch was not taken."""
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


def _settle(ctx, monkeypatch):
    """Whatever failures earlier tests forced are no longer held against the context."""
    monkeypatch.setenv("DP_SMALL", "1")
    dims = (4, 4, 4, 4)
    b = torch.ones(1, 256, 1, dtype=torch.complex128, device="cuda")
    for _ in range(257):
        ctx.solve_batch([ctx.operator(dims, 1, 0.5)], [b], ctx.opts())


@pytest.mark.parametrize("dims,n,block", [((8, 8, 8, 9), 18, 0), ((8, 8, 8, 9), 24, 32),  # three groups of four lanes
                                          ((7, 7, 7, 7), 29, 0), ((5, 5, 5, 5), 119, 128),  # six, 25: two rounds
                                          ((12, 8, 8, 8), 20, 32),   # one round of five groups, padding above
                                          ((8, 8, 4, 4), 4, 64), ((4, 3, 4, 5), 1, 256)])     # mostly padding
def test_rounds_match_oracle(ctx, monkeypatch, dims, n, block):
    _say("small rounds", dims, n, block)
    _settle(ctx, monkeypatch)
    rng = np.random.default_rng(8)
    N = int(np.prod(dims))
    U = workloads.random_links(dims, 0.4, 6)
    B = rng.standard_normal((n, N, 3)) + 1j * rng.standard_normal((n, N, 3))
    op = ctx.operator(dims, 3, 0.2, cuda(U))
    o = ctx.opts(tol=1e-12, rhs_block=block)
    got = {}
    for small in ("0", "1"):
        monkeypatch.setenv("DP_SMALL", small)
        (X,), (st,) = ctx.solve_batch([op], [cuda(B)], o)
        assert st["nconverged"] == st["nrhs"] == n
        got[small] = X
    assert not torch.equal(got["0"], got["1"])
    (X2,), _ = ctx.solve_batch([op], [cuda(B)], o)
    assert torch.equal(got["1"], X2)
    Xo, _, _ = oracle.cg_many(dims, 3, 0.2, U, B, tol=1e-14)
    assert np.abs(X2.cpu().numpy() - Xo).max() < 1e-10 * np.abs(Xo).max()


@pytest.mark.parametrize("dims,ns,block", [((8, 8, 8, 9), 8, 32),     # two rounds
                                           ((8, 8, 8, 8), 67, 8),      # 26 blocks of one round
                                           ((4, 4, 6, 4), 1, 64), ((5, 4, 3, 4), 2, 32)])  # mostly padding
def test_probes_and_gradients(ctx, monkeypatch, dims, ns, block):
    """Dense probes: the estimates, and the gradients, which sum over every lane
    of a block, against the launched kernels' (1e-10 of the largest)."""
    _say("small rounds, probes", dims, ns, block)
    _settle(ctx, monkeypatch)
    U = workloads.random_links(dims, 0.4, 3)
    op = ctx.operator(dims, 3, 0.3, cuda(U))
    ps = ctx.probe_spec(dims, 3, cuda(np.zeros(int(np.prod(dims)), np.int32)), 1, 5, 0, ns, "z2_complex", True)
    o = ctx.opts(tol=1e-12, rhs_block=block)
    got = {}
    for small in ("0", "1"):
        monkeypatch.setenv("DP_SMALL", small)
        T, g, dU, dUb, _ = ctx.trace_grad(op, ps, 1, o)
        got[small] = (ctx.trace_estimate([op], [ps], [1], o)[0]["tj"], dU.cpu().numpy(), dUb.cpu().numpy(),
                      np.array([T, g]))
    assert not np.array_equal(got["0"][0], got["1"][0])
    for a, b in zip(got["1"], got["0"]):
        assert np.abs(a - b).max() < 1e-10 * np.abs(b).max()


@pytest.mark.parametrize("dims,n,block", [((18, 12, 12, 12), 4, 4), ((16, 16, 16, 8), 2, 2), ((18, 12, 12, 12), 11, 4)])
def test_short_ring(ctx, monkeypatch, dims, n, block):
    """Without allocations the ring of the steps' vectors has as many slots as the
    fixed workspace leaves (four and seven here; four is the fewest that a solve that fits
    can get), so that it wraps more often: bit for bit the solve with eight."""
    _say("short ring", dims, n, block)
    _settle(ctx, monkeypatch)
    rng = np.random.default_rng(2)
    N = int(np.prod(dims))
    B = cuda(rng.standard_normal((n, N, 3)) + 1j * rng.standard_normal((n, N, 3)))
    op = ctx.operator(dims, 3, 0.1, cuda(workloads.random_links(dims, 0.4, 6)))
    o = ctx.opts(tol=1e-11, rhs_block=block)
    (X,), (st,) = ctx.solve_batch([op], [B], o)
    for _ in range(3):
        Y, sy = ctx.solve_noalloc(op, B, o)
        assert torch.equal(X, Y) and sy["rhs_iters"] == st["rhs_iters"] and sy["nconverged"] == n
    monkeypatch.setenv("DP_SMALL", "0")
    Z, _ = ctx.solve_noalloc(op, B, o)
    assert not torch.equal(X, Z) and (X - Z).abs().max() < 1e-9 * Z.abs().max()
