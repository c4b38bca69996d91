"""The Gram products of the deflation (FP64 matrix instruction, 32 x 32 output
tiles of 16-wide halves, 16 rows a turn): subspaces of 8 to 64 vectors and
right-hand-side blocks of 1 to 64, so that tiles are part filled, exactly
filled and several, over 1080 rows (two row ranges of 540, 12 more than a
whole number of turns).  Ritz values against a dense eigensolver (a Ritz value
is off by at most its residual, 1e-9 of itself asked for: bar 1e-8), and the
deflated contractions against dense algebra with the library's own vectors
(the split is exact for any vectors): |dt| <= |z| tol |b| / m2 with |b| at most
a few |z| against |z|^2 / (m2 + 8), below 1e-10 of it at tol 1e-12, m2 0.3."""
import sys

import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2106_01275_amd as dp  # noqa: E402


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return dp.context(0)


@pytest.mark.parametrize("nvec,blocks", [(1, (1, 16)), (6, (4, 64)), (20, (32, 8)), (40, (64, 16))])
def test_gram_tiles(ctx, nvec, blocks):
    print("gram tiles", nvec, blocks, flush=True)
    sys.stdout.flush()
    dims, m2, kind = (6, 5, 4, 3), 0.3, oracle.Z2_COMPLEX
    U = workloads.random_links(dims, 0.4, 12)
    op = ctx.operator(dims, 3, m2, torch.from_numpy(np.ascontiguousarray(U)).cuda())
    w, _ = oracle.lowest_eigenpairs(dims, 3, m2, U, nvec)
    d = ctx.deflation(op, nvec, tol=1e-9, seed=3)
    assert np.max(np.abs(d.evals - w[:nvec]) / w[:nvec]) < 1e-8
    V = d.vectors().cpu().numpy()
    assert np.abs(V.reshape(nvec, -1).conj() @ V.reshape(nvec, -1).T - np.eye(nvec)).max() < 1e-11
    col, m, _ = oracle.coloring(dims, 1, 1, oracle.NATURAL)
    ps = ctx.probe_spec(dims, 3, torch.from_numpy(np.ascontiguousarray(col)).cuda(), m, 9, 0, 2, "z2_complex", True)
    ref = oracle.trace_deflated(dims, 3, m2, U, 1, col, m, 9, 0, 2, kind, True, V)["tj"]
    scale = (np.abs(oracle.probes(dims, 3, col, m, 9, 0, 2, kind, True)) ** 2).sum((1, 2)) / (m2 + 8)
    for block in blocks:
        r = ctx.trace_deflated(op, d, 1, ps, ctx.opts(tol=1e-12, inner="f64", rhs_block=block))
        assert (np.abs(r["tj"] - ref) / scale).max() < 1e-10, block
    d.close()
