"""FP64 solves take every x update by itself, whatever the pairing option: the
same bits with and without it, in the single-instance and the multi-instance
engine, and solutions to the last digits.  The bar is an FP64 CG's own: its
recursive residual follows the true one to a few units of 2^-53 times the
condition number (A's norm is at most 16 + m2, its smallest eigenvalue at least
m2) per step, here below 30 steps of 32 units."""
import sys

import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2106_01275_amd as dp  # noqa: E402


@pytest.mark.parametrize("dims,nc", [((6, 6, 6, 6), 1), ((8, 4, 6, 4), 3), ((5, 4, 7, 3), 3)])
def test_x_updates_one_by_one(monkeypatch, dims, nc):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("fp64 updates", dims, nc, flush=True)
    sys.stdout.flush()
    ctx = dp.context(0)
    monkeypatch.setenv("DP_SMALL", "0")
    n, N, m2 = 12, int(np.prod(dims)), 0.5
    U = workloads.random_links(dims, 0.3, 3, nc) if nc == 3 else None
    cuda = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    rng = np.random.default_rng(1)
    B = rng.choice([-1.0, 1.0], (n, N, nc)) + 1j * rng.choice([-1.0, 1.0], (n, N, nc))
    op = ctx.operator(dims, nc, m2, None if U is None else cuda(U))
    o = ctx.opts(tol=1e-15, inner="f64", rhs_block=16)
    got = {}
    for pairs in ("0", "1"):
        monkeypatch.setenv("DP_XDEFER", pairs)
        got[pairs] = [x for k in (1, 2) for x in ctx.solve_batch([op] * k, [cuda(B)] * k, o, check=False)[0]]
    for a, b in zip(got["0"], got["1"]):
        assert torch.equal(a, b)
    Xo, _, _ = oracle.cg_many(dims, nc, m2, U, B, tol=1e-15)
    bar = 2 * 30 * 32 * 2.0 ** -53 * (16 + m2) / m2
    for x in got["1"]:
        err = (x.cpu().numpy() - Xo).reshape(n, -1)
        assert (np.linalg.norm(err, axis=1) <= bar * np.linalg.norm(Xo.reshape(n, -1), axis=1)).all()
