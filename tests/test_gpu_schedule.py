"""The schedule of the launched single-instance solves away from well
conditioned operators.

A free field of small mass (condition number of the reduced system 80 at m2 =
0.05, 400 at 0.01): FP32 keeps to the FP64 solve's number of iterations, as
FP64-accurate CG would, with a little for what its rounding and its updates
cost: an update loses about two steps (four iterations), three are due to 1e-10,
and a check comes up to eight steps after the tolerance is met.  Bar: a quarter
more, and 16, for right-hand sides with the whole spectrum.  (A smooth one's
Krylov space is small, and FP32's loss of conjugacy in it costs half as many
iterations again under any schedule: there the result alone is held.)

reliable_delta, given by the caller, sets the drop between FP32's updates: a
check falls on the predicted step, at most one step late of a decay of about a
digit a step, so an update gains at least the drop asked for and at most about
two digits more."""
import math
import sys

import numpy as np
import pytest

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


def _rhs(kind, n, N, nc, seed):
    rng = np.random.default_rng(seed)
    if kind == "noise":
        return rng.choice([-1.0, 1.0], (n, N, nc)) + 1j * rng.choice([-1.0, 1.0], (n, N, nc))
    return np.ones((n, N, nc), complex) + 0.1 * rng.standard_normal((n, N, nc))


@pytest.mark.parametrize("m2", [0.05, 0.01])
@pytest.mark.parametrize("kind", ["noise", "smooth"])
@pytest.mark.parametrize("dims", [(16, 16, 16, 16), (15, 12, 10, 14)])
def test_fp32_on_light_operators(ctx, monkeypatch, dims, kind, m2):
    _say("light", dims, kind, m2)
    monkeypatch.setenv("DP_SMALL", "0")
    op = ctx.operator(dims, 1, m2, None)
    B = cuda(_rhs(kind, 12, int(np.prod(dims)), 1, 3))
    for block in (1, 4, 16):  # twelve blocks, three, one
        (X,), (s64,) = ctx.solve_batch([op], [B], ctx.opts(tol=1e-10, inner="f64", rhs_block=block))
        (Y,), (s32,) = ctx.solve_batch([op], [B], ctx.opts(tol=1e-10, inner="f32", rhs_block=block))
        _say("  ", block, s64["rhs_iters"] / 12, s32["rhs_iters"] / 12, s32["reliable_updates"])
        assert s32["nconverged"] == 12 and s32["max_true_resid"] <= 1e-10
        # |dx| <= (tol_1 + tol_2) |b| / m2
        assert ((X - Y).flatten(1).norm(dim=1) <= 3e-10 / m2 * B.flatten(1).norm(dim=1)).all()
        if kind == "noise":
            assert s32["rhs_iters"] <= 1.25 * s64["rhs_iters"] + 16 * 12, block


@pytest.mark.parametrize("dims", [(8, 8, 8, 8), (8, 7, 8, 5)])
def test_fp32_drop_is_the_callers(ctx, monkeypatch, dims):
    _say("drop", dims)
    monkeypatch.setenv("DP_SMALL", "0")
    U = workloads.random_links(dims, 0.4, 6)
    op = ctx.operator(dims, 3, 0.1, cuda(U))
    B = cuda(_rhs("noise", 8, int(np.prod(dims)), 3, 4))
    for delta in (0.1, 0.01, 1e-4):
        _, (st,) = ctx.solve_batch([op], [B], ctx.opts(tol=1e-11, inner="f32", rhs_block=8, reliable_delta=delta))
        _say("  ", delta, st["reliable_updates"])
        assert st["nconverged"] == 8
        digits = -math.log10(delta)
        assert math.ceil(11 / (digits + 2)) <= st["reliable_updates"] <= math.ceil(11 / digits) + 1, delta


@pytest.mark.parametrize("dims,eps", [((16, 8, 8, 8), 0), ((4, 4, 4, 4), 0), ((5, 4, 3, 4), 0), ((4, 3, 2, 4), 0.3)])
def test_exhausted_krylov_space(ctx, monkeypatch, dims, eps):
    """FP32 where a handful of steps solves a system exactly (a few plane waves of
    the free field, lattices of few sites): the recursive residual falls below
    what FP32 resolves, and a lane whose residual then grows starts again from the
    true one.  Every right-hand side converges, well before the limit (the true
    residual is the library's own, in FP64)."""
    _say("exhausted", dims)
    monkeypatch.setenv("DP_SMALL", "0")
    N, n = int(np.prod(dims)), 6
    ix = np.indices(dims)
    for seed in range(12):
        U = workloads.random_links(dims, eps, seed, 1) if eps else None
        for m2 in (0.02, 0.3):
            op = ctx.operator(dims, 1, m2, None if U is None else cuda(U))
            rng = np.random.default_rng(seed)
            B = rng.choice([-1.0, 1.0], (n, N, 1)) + 1j * rng.choice([-1.0, 1.0], (n, N, 1))
            for j in range(3):
                B[j] = 0
                for _ in range(j + 1 + seed % 4):
                    k = [rng.integers(d) for d in dims]
                    B[j] += (rng.standard_normal() * np.exp(2j * np.pi * sum(a * x / d for a, x, d in zip(k, ix, dims)))
                             ).reshape(N, 1)
            B[4] *= rng.random((N, 1)) < 0.15
            if not np.abs(B[4]).any():
                B[4][0] = 1
            for block in (1, 8):
                _, (st,) = ctx.solve_batch([op], [cuda(B)], ctx.opts(tol=1e-10, inner="f32", rhs_block=block, max_iter=1500),
                                           check=False)
                assert st["nconverged"] == n and st["max_true_resid"] <= 1e-10, (seed, m2, block)
