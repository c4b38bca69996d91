"""The numbered sums of the persistent solves: their numbers start over (over
cleared words) when the launches of a context have used them up, which a large
iteration limit brings about at once, since a launch sets aside what its limit
could use.  In the order of the call's stream, whichever that is."""
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


@pytest.mark.parametrize("limit", [200_000_000, 700_000_000, 2 ** 31 - 1])  # every few launches, two, every one
@pytest.mark.parametrize("dims", [(8, 4, 4, 6), (5, 4, 3, 6)])
def test_numbers_start_over(ctx, monkeypatch, limit, dims):
    """A queue of a dozen and more blocks, on the default stream, a side stream
    and the library's own: bit for bit as with the default limit."""
    _say("small sums", limit, dims)
    monkeypatch.setenv("DP_SMALL", "1")
    U = workloads.random_links(dims, 0.4, 3)
    col, m, _ = oracle.coloring(dims, 1, 2, oracle.NATURAL)
    op = ctx.operator(dims, 3, 0.3, cuda(U))
    ps = ctx.probe_spec(dims, 3, cuda(col), m, 5, 0, 2, "z2_complex", True)
    ref = ctx.trace_estimate([op], [ps], [1], ctx.opts(tol=1e-11, rhs_block=4))[0]
    assert ref["solve"]["nrhs"] > 48
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    for turn in range(3):
        for stream, graph in ((torch.cuda.current_stream(), 0), (side, 0), (side, 1)):
            with torch.cuda.stream(stream):
                t = ctx.trace_estimate([op], [ps], [1], ctx.opts(tol=1e-11, rhs_block=4, max_iter=limit,
                                                                 use_graph=graph))[0]
            assert np.array_equal(t["tj"], ref["tj"]) and t["solve"]["rhs_iters"] == ref["solve"]["rhs_iters"]
