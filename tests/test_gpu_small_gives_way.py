"""Persistent solves that give up (their waits run out, here because no polls
are allowed from some launch of a call on): the call is finished by the
launched kernels, whatever it had done by then."""
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


@pytest.fixture(scope="module")
def problem(ctx):
    dims, n = (6, 4, 4, 4), 10
    rng = np.random.default_rng(4)
    U = workloads.random_links(dims, 0.4, 3)
    B = rng.standard_normal((n, 384, 3)) + 1j * rng.standard_normal((n, 384, 3))
    Xo, _, _ = oracle.cg_many(dims, 3, 0.2, U, B, tol=1e-14)
    return dims, U, B, Xo


@pytest.mark.parametrize("inner", ["f64", "f32"])
@pytest.mark.parametrize("first", [0, 1, 2])
def test_in_place_solve_goes_on(ctx, problem, monkeypatch, inner, first):
    """x in b's own memory, three blocks of at most four right-hand sides, the
    first, second or third gives up: the x already written are not solved for
    again.  To the bars of the other solve tests (1e-10 at a residual of 1e-12,
    1e-8 at 1e-10); every right-hand side is counted once."""
    _say("in place", inner, first)
    dims, U, B, Xo = problem
    op = ctx.operator(dims, 3, 0.2, cuda(U))
    o = ctx.opts(tol=1e-12 if inner == "f64" else 1e-10, inner=inner, rhs_block=4)
    monkeypatch.setenv("DP_SMALL", "1")
    for call in ("solve_batch", "solve_noalloc"):
        X = cuda(B)
        monkeypatch.setenv("DP_SMALL_POLLS", f"0:{first}")
        if call == "solve_batch":
            _, (st,) = ctx.solve_batch([op], [X], o, xs=[X])
        else:
            _, st = ctx.solve_noalloc(op, X, o, x=X)
        monkeypatch.delenv("DP_SMALL_POLLS")
        assert st["nrhs"] == st["nconverged"] == len(B)
        err = np.abs(X.cpu().numpy() - Xo).max() / np.abs(Xo).max()
        assert err < (1e-10 if inner == "f64" else 1e-8), (call, err)
