"""The even-odd reduction behind the solves on lattices whose extents are all
even, in plain numpy on the oracle's operator: hops connect sites of opposite
parity only, and x_e from S x_e = b_e + H b_o / c, S = c - H H / c, with
x_o = (b_o + H x_e) / c solves A x = b; the residual of any x_e with that x_o
is the reduced system's, on the even sites alone (so a stopping rule relative
to |b| means the same).  The internal order, parity * N / 2 + index / 2, is a
permutation whose halves keep the index order."""
import numpy as np
import pytest

import oracle
import workloads


@pytest.mark.parametrize("dims,nc,links", [((2, 2, 2, 2), 3, True), ((4, 2, 2, 6), 1, True), ((2, 4, 4, 2), 1, False),
                                           ((4, 2, 4, 2), 3, True)])
def test_reduction(dims, nc, links):
    m2, N = 0.3, int(np.prod(dims))
    c = m2 + 8.0
    U = workloads.random_links(dims, 0.5, 3, nc) if links else None
    n = N * nc
    A = np.stack([oracle.apply(dims, nc, m2, U, e.reshape(N, nc)).ravel() for e in np.eye(n, dtype=complex)], 1)
    parity = np.indices(dims).sum(0).ravel() % 2
    p = np.repeat(parity, nc)
    H = c * np.eye(n) - A
    e, o = p == 0, p == 1
    assert np.abs(H[np.ix_(e, e)]).max() == 0 and np.abs(H[np.ix_(o, o)]).max() == 0
    rng = np.random.default_rng(1)
    b = rng.standard_normal(n) + 1j * rng.standard_normal(n)
    S = c * np.eye(e.sum()) - H[np.ix_(e, o)] @ H[np.ix_(o, e)] / c
    x = np.zeros(n, complex)
    x[e] = np.linalg.solve(S, b[e] + H[np.ix_(e, o)] @ b[o] / c)
    x[o] = (b[o] + H[np.ix_(o, e)] @ x[e]) / c
    assert np.abs(A @ x - b).max() < 1e-12
    x[e] += 1e-3 * rng.standard_normal(e.sum())
    x[o] = (b[o] + H[np.ix_(o, e)] @ x[e]) / c
    r = b - A @ x
    red = b[e] + H[np.ix_(e, o)] @ b[o] / c - S @ x[e]
    assert np.abs(r[o]).max() < 1e-13 and np.abs(r[e] - red).max() < 1e-13
    # c > 0: A is positive definite exactly when S is
    for shift in (0.0, np.linalg.eigvalsh(A)[0] - 0.05):
        cs = c - shift
        if cs > 0:
            Ss = cs * np.eye(e.sum()) - H[np.ix_(e, o)] @ H[np.ix_(o, e)] / cs
            assert (np.linalg.eigvalsh(A - shift * np.eye(n))[0] > 0) == (np.linalg.eigvalsh(Ss)[0] > 0)
    order = parity * (N // 2) + np.arange(N) // 2
    assert np.array_equal(np.sort(order), np.arange(N))
    inv = np.argsort(order)
    assert np.all(np.diff(inv[: N // 2]) > 0) and np.all(np.diff(inv[N // 2:]) > 0)
