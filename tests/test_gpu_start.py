"""The start of a block in even-odd order (launched kernels): probes enter as
r = p = b_e + H b_o / c, formed where the probes are nonzero, and the solution is
first written by its first fold.  Against the oracle's estimates: extents of 2,
colours on both parities and on one site each, dense probes, every kind of
noise, every kind of block width (one right-hand side, a tile of many sites, a
wavefront and more per site), a last block with idle lanes, and several blocks
per call on stale scratch.  An estimate's error is at most |v| |dx| with
|dx| <= tol |v| / m2, against values of about |v|^2 / (m2 + 8): 8.3 tol / m2 of
them, below 1e-10 at FP64's 1e-12 and 1e-8 at 1e-10 for m2 = 0.3."""
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


CASES = [((2, 2, 2, 2), 3, True, "z2_complex", True, 1, 1), ((2, 2, 2, 2), 1, False, "real_z2", False, 2, 8),
         ((4, 2, 6, 2), 3, True, "z4", False, 3, 2), ((6, 4, 2, 10), 3, True, "z2_complex", True, 2, 16),
         ((8, 2, 4, 6), 1, True, "z4", False, 40, 32), ((16, 2, 2, 4), 3, True, "real_z2", True, 2, 64),
         ((8, 4, 4, 2), 3, False, "z2_complex", True, 3, 128), ((4, 4, 2, 4), 3, True, "z4", True, 9, 256)]


_REF = {}


@pytest.mark.parametrize("dims,nc,links,noise,dilute,ns,block", CASES)
@pytest.mark.parametrize("inner", ["f64", "f32", "bf16"])
def test_probe_start_matches_oracle(ctx, monkeypatch, inner, dims, nc, links, noise, dilute, ns, block):
    print("probe start", inner, dims, nc, links, noise, dilute, ns, block, flush=True)
    sys.stdout.flush()
    monkeypatch.setenv("DP_SMALL", "0")
    kind = {"real_z2": 0, "z2_complex": 1, "z4": 2}[noise]
    N = int(np.prod(dims))
    U = workloads.random_links(dims, 0.4, 7, nc) if links else None
    op = ctx.operator(dims, nc, 0.3, None if U is None else cuda(U))
    o = ctx.opts(tol=1e-12 if inner == "f64" else 1e-10, inner=inner, rhs_block=block)
    parity = np.indices(dims).sum(0).ravel() % 2
    for col, m in ((np.zeros(N, np.int32), 1),                    # dense probes
                   ((np.arange(N) % 5).astype(np.int32), 5),      # both parities in a colour
                   ((parity * 2 + np.arange(N) // 2 % 2).astype(np.int32), 4),
                   (np.arange(N).astype(np.int32), N)):           # one site per colour
        s = 1 if m == N else ns
        ps = ctx.probe_spec(dims, nc, cuda(col), m, 11, 2, s, noise, dilute)
        key = (dims, nc, m)
        if key not in _REF:
            _REF[key] = (oracle.trace(dims, nc, 0.3, U, 1, col, m, 11, 2, s, kind, dilute, tol=1e-14)["tj"],
                         (np.abs(oracle.probes(dims, nc, col, m, 11, 2, s, kind, dilute)) ** 2).sum((1, 2)) / 8.3)
        ref, scale = _REF[key]
        for call in ("single", "batch"):
            k = 1 if call == "single" else 2
            for r in ctx.trace_estimate([op] * k, [ps] * k, [1] * k, o):
                err = (np.abs(r["tj"] - ref)[scale > 0] / scale[scale > 0]).max()
                assert np.all(r["tj"][scale == 0] == 0)
                assert err < (1e-10 if inner == "f64" else 1e-8), (call, m, err)


@pytest.mark.parametrize("dims", [(4, 4, 2, 4), (4, 3, 2, 5)])
@pytest.mark.parametrize("inner", ["f32", "bf16"])
def test_zero_rhs_after_a_solve(ctx, monkeypatch, inner, dims):
    """A block without an active lane is never updated: its solution is zero
    all the same, whatever the scratch held before."""
    monkeypatch.setenv("DP_SMALL", "0")
    N = int(np.prod(dims))
    rng = np.random.default_rng(3)
    B = cuda(rng.standard_normal((6, N, 3)) + 1j * rng.standard_normal((6, N, 3)))
    op = ctx.operator(dims, 3, 0.3, cuda(workloads.random_links(dims, 0.4, 7)))
    o = ctx.opts(tol=1e-10, inner=inner, rhs_block=8)
    for k in (1, 3):
        Xs, _ = ctx.solve_batch([op] * k, [B] * k, o)
        assert all(float(x.abs().max()) > 0 for x in Xs)
        Zs, sts = ctx.solve_batch([op] * k, [torch.zeros_like(B)] * k, o)
        assert all(torch.all(z == 0) for z in Zs) and all(s["nconverged"] == 6 for s in sts)
