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


@pytest.mark.parametrize("first", [0, 7])
def test_queued_launches_give_way(ctx, monkeypatch, first):
    """Estimates whose blocks are queued one behind the other (a trace, every
    level's adjoint, deflated probes): the first or the eighth launch gives up,
    those behind it end at once, and the call's results are the launched
    kernels' own, as are the next calls' to the bars of the tolerance (1e-10 of
    the largest)."""
    _say("queue", first)
    dims = (4, 4, 6, 4)
    U = workloads.random_links(dims, 0.4, 3)
    col, m, _ = oracle.coloring(dims, 1, 2, oracle.NATURAL)
    op = ctx.operator(dims, 3, 0.3, cuda(U))
    ps = ctx.probe_spec(dims, 3, cuda(col), m, 5, 0, 2, "z2_complex", True)
    o = ctx.opts(tol=1e-12, rhs_block=2)
    d = ctx.deflation(op, 6, tol=1e-8, seed=2)
    calls = (lambda: ctx.trace_estimate([op], [ps], [1], o)[0]["tj"],
             lambda: np.concatenate([np.ravel(v.cpu().numpy() if torch.is_tensor(v) else v)
                                     for v in ctx.trace_grad(op, ps, 1, o)[:4]]),
             lambda: ctx.trace_deflated(op, d, 1, ps, o)["tj"])
    for k, call in enumerate(calls):
        monkeypatch.setenv("DP_SMALL", "0")
        ref = call()
        monkeypatch.setenv("DP_SMALL", "1")
        before = call()
        monkeypatch.setenv("DP_SMALL_POLLS", f"0:{first}")
        got = call()
        monkeypatch.delenv("DP_SMALL_POLLS")
        assert np.array_equal(got, ref), k
        for after in (before, call(), call(), call()):
            assert np.abs(after - ref).max() < 1e-10 * np.abs(ref).max(), k
    d.close()


def test_failures_are_remembered(ctx, problem, monkeypatch):
    """Under lasting contention a context does not wait in every call: after a
    failure the next call that could take a persistent launch does not try, after
    a second one in a row the next two, and so on; a success ends that.  (The two
    paths round differently, so bits tell which one a call took.)"""
    _say("remembered")
    dims, U, B, _ = problem
    op, b = ctx.operator(dims, 3, 0.2, cuda(U)), cuda(B)
    o = ctx.opts(tol=1e-11, rhs_block=16)
    solve = lambda: ctx.solve_batch([op], [b], o)[0][0]  # noqa: E731
    monkeypatch.setenv("DP_SMALL", "0")
    launched = solve()
    monkeypatch.setenv("DP_SMALL", "1")
    for _ in range(256):  # (whatever calls before this test left)
        small = solve()
        if not torch.equal(small, launched):
            break
    took = lambda: "launched" if torch.equal(solve(), launched) else "small"  # noqa: E731
    assert took() == took() == "small" and torch.equal(solve(), small)
    for turn in range(2):  # (the second time as the first: the success between them ended the count)
        for skipped in (1, 2, 4):
            monkeypatch.setenv("DP_SMALL_POLLS", "0")
            assert took() == "launched"
            monkeypatch.delenv("DP_SMALL_POLLS")
            for _ in range(skipped):
                assert took() == "launched"
        assert took() == took() == "small"


@pytest.mark.parametrize("dims,n", [((8, 8, 8, 8), 8), ((9, 8, 7, 8), 7)])
def test_several_threads(ctx, monkeypatch, dims, n):
    """Four host threads, each with its own context and stream, solve at once.
    Persistent launches of two contexts can keep each other from becoming
    resident; the waits then run out and the launched kernels take the call.  The
    right solutions (1e-10 at 1e-12), and on the average of all calls at most 20
    ms: a wait that runs out is below 2 ms, the launched solves of four threads
    sharing the GPU below 2 ms each, and a call has at most one of each."""
    import threading
    import time

    _say("threads", dims, n)
    monkeypatch.setenv("DP_SMALL", "1")
    N = int(np.prod(dims))
    rng = np.random.default_rng(2)
    U = workloads.random_links(dims, 0.4, 3)
    B = rng.standard_normal((n, N, 3)) + 1j * rng.standard_normal((n, N, 3))
    Xo, _, _ = oracle.cg_many(dims, 3, 0.2, U, B, tol=1e-14)
    Ug, b = cuda(U), cuda(B)
    torch.cuda.synchronize()
    threads, calls = 4, 40
    start, errs, secs = threading.Barrier(threads), [], []

    def work():
        c = dp.Context(0)
        with torch.cuda.stream(torch.cuda.Stream()):
            op, o, x = c.operator(dims, 3, 0.2, Ug), c.opts(tol=1e-12), torch.empty_like(b)
            c.solve_batch([op], [b], o, xs=[x])
            start.wait()
            t = time.perf_counter()
            for _ in range(calls):
                x.zero_()
                _, (st,) = c.solve_batch([op], [b], o, xs=[x])
                errs.append(np.abs(x.cpu().numpy() - Xo).max() if st["nconverged"] == n else np.inf)
            secs.append(time.perf_counter() - t)
        c.close()

    pool = [threading.Thread(target=work) for _ in range(threads)]
    for p in pool:
        p.start()
    for p in pool:
        p.join()
    assert len(errs) == threads * calls and max(errs) < 1e-10 * np.abs(Xo).max()
    _say("   ms a call", 1e3 * sum(secs) / (threads * calls))
    assert sum(secs) / (threads * calls) < 20e-3
