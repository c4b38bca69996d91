"""Performance cases of the library's public entry points.

Every case is one call that a program using the library makes: a probed trace,
an adjoint gradient, a batch of linear solves, many uneven instances in one
call, through the Python binding, from the tiny free field that is all launch
latency to the 32^4 lattice whose vectors fill the memory system.  The
lattices, masses, link roughness, displacements and distances are those of
workloads.py and the tests, or lie between them.

Solves run to relative residuals of 1e-11 .. 1e-12 (the tests' range), so that
an output is fixed by its inputs to about ten digits and not by the iteration
at which a solver happens to stop.

A case is a dict:
  kind    "trace"    Context.trace_estimate of one lattice
          "multi"    Context.trace_multi: displacements 0 .. p from one set of solves
          "deflated" Context.trace_deflated (the deflation vectors are kept by the caller)
          "batch"    Context.trace_estimate of ninst lattices in one call
          "grad"     Context.trace_grad: T, dT/dm2 and the link gradients
          "autograd" probed_trace and backward() of a real loss
          "solve"    Context.solve_batch with nrhs dense right-hand sides
          "noalloc"  Context.solve_noalloc, the same without device allocations
          "apply"    Context.apply: A v for nrhs vectors
  d0..d3  lattice extents; nc colours per site (1: free field, 3: random links)
  m2, eps mass term and link roughness, U = exp(i eps H)
  p, k    displacement and distance of the colouring; order its visitation order
  ns      noise samples; noise its kind; dilute whether colour is diluted
  inner   storage precision of the solver; tol its relative residual
  block   right-hand sides per block (0: the library chooses)
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

import paper_2106_01275_amd as dp

NORM = dp.NOISE_NORM


def listed():
    return [
        # the smallest call there is: a 4^4 free field, one block of eight
        # right-hand sides (launches and host round trips only)
        dict(name="trace-free4-f64", kind="trace", d0=4, d1=4, d2=4, d3=4, nc=1, m2=0.5, eps=0.0, p=1, k=2,
             order="best", ns=1, noise="real_z2", dilute=False, inner="f64", tol=1e-12, block=0),
        # one propagator column on a small gauge lattice: latency of a single solve
        dict(name="solve8-one-f64", kind="solve", d0=8, d1=8, d2=8, d3=8, nc=3, m2=0.1, eps=0.3, nrhs=1,
             inner="f64", tol=1e-12, block=0),
        # a handful of sources in a serving loop that must not allocate
        dict(name="noalloc8-f32", kind="noalloc", d0=8, d1=8, d2=8, d3=8, nc=3, m2=0.1, eps=0.3, nrhs=20,
             inner="f32", tol=1e-11, block=0),
        # the small gauge workload in the library's default precision: one
        # diluted sample, 192 right-hand sides
        dict(name="trace8-f64", kind="trace", d0=8, d1=8, d2=8, d3=8, nc=3, m2=0.1, eps=0.3, p=2, k=4,
             order="best", ns=1, noise="z2_complex", dilute=True, inner="f64", tol=1e-12, block=0),
        # odd extents and a ragged last block
        dict(name="solve-odd-f32", kind="solve", d0=9, d1=10, d2=7, d3=12, nc=3, m2=0.15, eps=0.4, nrhs=45,
             inner="f32", tol=1e-11, block=0),
        # the finest level of the nested 16^4 workload: 960 colours x 3
        # dilutions, the throughput case
        dict(name="trace16-fine-f32", kind="trace", d0=16, d1=16, d2=16, d3=16, nc=3, m2=0.05, eps=0.4, p=4, k=8,
             order="nested", ns=1, noise="z2_complex", dilute=True, inner="f32", tol=1e-11, block=0),
        # the level that reaches a given error soonest, with BF16 storage, and
        # every displacement from one set of solves
        dict(name="multi16-bf16", kind="multi", d0=16, d1=16, d2=16, d3=16, nc=3, m2=0.05, eps=0.4, p=4, k=4,
             order="natural", ns=4, noise="z2_complex", dilute=True, inner="bf16", tol=1e-11, block=0),
        # 64 uneven lattices in one call
        dict(name="batch64-bf16", kind="batch", ninst=64, shapes=4, nc=3, k=4, ns=1, noise="z2_complex", dilute=True,
             inner="bf16", tol=1e-11, block=0),
        # a few lattices in the default precision
        dict(name="batch9-f64", kind="batch", ninst=9, shapes=7, nc=3, k=2, ns=2, noise="z4", dilute=False,
             inner="f64", tol=1e-12, block=0),
        # trace and adjoint gradient of the largest lattice (a short displacement:
        # at long ones the gradient is a small remainder of large terms)
        dict(name="grad32-f32", kind="grad", d0=32, d1=32, d2=32, d3=32, nc=3, m2=0.01, eps=0.5, p=2, k=3,
             order="natural", ns=2, noise="z2_complex", dilute=True, inner="f32", tol=1e-12, block=0),
        # a differentiable estimate inside an optimisation loop: forward and
        # backward through torch.autograd
        dict(name="autograd8-f64", kind="autograd", d0=8, d1=8, d2=8, d3=8, nc=3, m2=0.2, eps=0.5, p=1, k=2,
             order="best", ns=2, noise="z2_complex", dilute=True, inner="f64", tol=1e-12, block=0),
        # low modes deflated, the probes estimate the rest
        dict(name="deflated16-f32", kind="deflated", d0=16, d1=16, d2=16, d3=16, nc=3, m2=0.05, eps=0.4, p=1, k=2,
             order="natural", ns=4, noise="z2_complex", dilute=True, inner="f32", tol=1e-11, block=0, nvec=12),
    ]


# ------------------------------------------------------------------ sizes


def _dims(case):
    return (case["d0"], case["d1"], case["d2"], case["d3"])


@functools.lru_cache(maxsize=None)
def _colouring(dims, p, k, order):
    """A program colours a lattice once and keeps it.  "nested": the finest of
    the levels 1, 2, 4, .. k."""
    if order == "nested":
        ks = [d for d in (1, 2, 4, 8) if d <= k]
        col, n, _ = dp.build_coloring(dims, p, ks, "natural")
        return np.ascontiguousarray(col[-1]), int(n[-1])
    col, n, _ = dp.build_coloring(dims, p, k, order)
    return np.ascontiguousarray(col), int(n)


@functools.lru_cache(maxsize=None)
def _instances(ninst, shapes):
    """(dims, m2, eps, p) of an uneven batch: extents from {4, 6, 8, 10, 12},
    masses, roughness and displacements drawn from PCG64(shapes)."""
    rng = np.random.Generator(np.random.PCG64(shapes))
    out = []
    for _ in range(ninst):
        dims = tuple(int(v) for v in rng.choice([4, 6, 8, 10, 12], size=4))
        out.append((dims, float(rng.uniform(0.05, 0.5)), float(rng.uniform(0.2, 0.5)), int(rng.choice([1, 2, 3]))))
    return tuple(out)


def _probe_count(case, dims, p):
    _, m = _colouring(dims, p, case["k"], case.get("order", "best"))
    return case["ns"] * m * (case["nc"] if case["dilute"] else 1)


def _parts(case):
    """[(sites, right-hand sides solved)] of a case."""
    if case["kind"] == "batch":
        return [(math.prod(d), _probe_count(case, d, p)) for d, _, _, p in _instances(case["ninst"], case["shapes"])]
    n = math.prod(_dims(case))
    if "nrhs" in case:
        return [(n, case["nrhs"])]
    r = _probe_count(case, _dims(case), case["p"])
    # the gradient solves the adjoint systems too; autograd also solves the
    # forward ones a second time in its backward pass
    return [(n, r * {"grad": 2, "autograd": 3}.get(case["kind"], 1))]


def work(case):
    """Every solve applies the operator about ln(2 / tol) / 1.1 times (the best
    polynomial at the condition number of about 14 that these lattices have);
    an application reads and writes a vector of the storage precision and does
    eight colour-matrix products a site.  The links are read once, and the
    vectors at the interface once."""
    nc, size = case["nc"], {"f64": 16, "f32": 8, "bf16": 4}[case["inner"]]
    links = 16 * 4 * nc * nc if nc == 3 else 0
    applies = 1 if case["kind"] == "apply" else math.ceil(math.log(2 / case["tol"]) / 1.1)
    b = f = 0.0
    for n, r in _parts(case):
        b += n * links + n * r * nc * 2 * size * applies
        f += n * r * applies * (8 * 8 * nc * nc if nc == 3 else 16)
        if "nrhs" in case:
            b += n * r * nc * 32
        if case["kind"] in ("grad", "autograd"):
            b += 2 * n * 16 * 4 * nc * nc
    return {"bytes": b, "flops": f}


def draw(rng):
    """One more case of the listed ranges: the kinds above on lattices from
    4^4 to 16^4 (extents from 3 up, odd ones among them), one to a few hundred
    right-hand sides."""
    kind = rng.choice(["trace", "trace", "multi", "batch", "grad", "autograd", "solve", "solve", "noalloc",
                       "deflated", "apply"])
    inner = rng.choice(["f64", "f32", "bf16"])
    c = dict(kind=kind, nc=3, inner=inner, tol=1e-12 if inner == "f64" else 1e-11, block=0)
    if kind == "batch":
        return dict(c, ninst=rng.randint(2, 40), shapes=rng.randint(100, 100000), k=rng.choice([1, 2, 3, 4]),
                    ns=rng.randint(1, 2), noise=rng.choice(["z4", "z2_complex"]), dilute=rng.random() < 0.7)
    while True:
        if rng.random() < 0.25:
            d = [rng.randint(3, 13) for _ in range(4)]
        else:
            d = [2 * rng.randint(2, 8) for _ in range(4)]
        n = math.prod(d)
        if n <= {"autograd": 8000, "noalloc": 2500, "batch": 0}.get(kind, 70000):
            break
    c.update(d0=d[0], d1=d[1], d2=d[2], d3=d[3], m2=round(rng.uniform(0.05, 0.5), 3), eps=round(rng.uniform(0.2, 0.5), 3))
    if kind in ("solve", "noalloc", "apply"):
        most = 20 if kind == "noalloc" else max(1, min(200, 6_000_000 // n))
        c["nrhs"] = max(1, round(math.exp(rng.uniform(0.0, math.log(most)))))
        if kind == "solve" and rng.random() < 0.2:
            c["block"] = rng.choice([1, 8, 16, 64])
        return c
    if kind in ("grad", "autograd"):
        c["tol"] = 1e-12
    c.update(p=rng.randint(0, 2 if kind in ("grad", "autograd") else 3), k=rng.choice([1, 2, 3, 4]), order=rng.choice(["natural", "best"]),
             ns=rng.randint(1, 3), noise=rng.choice(["real_z2", "z2_complex", "z4"]), dilute=rng.random() < 0.7)
    if kind == "deflated":
        c["nvec"] = rng.randint(4, 12)
    return c


# ------------------------------------------------------------------ inputs


def _links(dims, eps, g):
    """U = exp(i eps H), H traceless Hermitian from normal deviates
    (complex128 [4, N, 3, 3]): a Taylor series of exp(i eps H / 16) squared
    four times."""
    n = math.prod(dims)
    G = torch.randn((4, n, 3, 3, 2), generator=g, device="cuda", dtype=torch.float64)
    G = torch.view_as_complex(G)
    H = 0.5 * (G + G.transpose(-1, -2).conj())
    H = H - (torch.diagonal(H, dim1=-2, dim2=-1).sum(-1) / 3)[..., None, None] * torch.eye(3, device="cuda")
    X = 1j * (eps / 16) * H

    def mul(A, B):
        return sum(A[..., :, b, None] * B[..., b, None, :] for b in range(3))

    eye = torch.eye(3, device="cuda", dtype=torch.complex128).expand_as(X)
    E = eye
    for j in range(11, 0, -1):
        E = eye + mul(X, E) / j
    for _ in range(4):
        E = mul(E, E)
    return E.contiguous()


def _gen(seed, i=0):
    g = torch.Generator(device="cuda")
    g.manual_seed(1000003 * (seed + 1) + i)
    return g


def _lattice(case, dims, m2, eps, p, seed, i):
    """One lattice's operator and probes, as plain data."""
    s = {"dims": dims, "m2": m2, "p": p, "seed": seed * 131 + i,
         "U": _links(dims, eps, _gen(seed, i)) if case["nc"] == 3 else None}
    if "k" in case:
        col, m = _colouring(dims, p, case["k"], case.get("order", "best"))
        s["col"], s["m"] = torch.from_numpy(col).cuda(), m
    if "nrhs" in case:
        g = _gen(seed, 7777)
        s["b"] = torch.view_as_complex(torch.randn((case["nrhs"], math.prod(dims), case["nc"], 2), generator=g,
                                                   device="cuda", dtype=torch.float64))
    return s


def _data(case, seed):
    if case["kind"] == "batch":
        return [_lattice(case, d, m2, eps, p, seed, i)
                for i, (d, m2, eps, p) in enumerate(_instances(case["ninst"], case["shapes"]))]
    return [_lattice(case, _dims(case), case["m2"], case["eps"], case.get("p", 0), seed, 0)]


def prepare(case, seed):
    ctx = dp.context(0)
    data = _data(case, seed)
    s = {"kind": case["kind"], "ctx": ctx, "data": data, "inner": case["inner"], "p": [d["p"] for d in data],
         "opts": ctx.opts(tol=case["tol"], inner=case["inner"], rhs_block=case["block"]),
         "ops": [ctx.operator(d["dims"], case["nc"], d["m2"], d["U"]) for d in data]}
    if "k" in case:
        s["ps"] = [ctx.probe_spec(d["dims"], case["nc"], d["col"], d["m"], d["seed"], 0, case["ns"], case["noise"],
                                  case["dilute"]) for d in data]
    if case["kind"] == "deflated":
        s["defl"] = ctx.deflation(s["ops"][0], case["nvec"], tol=1e-6, seed=1, check=False)
    if case["kind"] == "autograd":
        d = data[0]
        s["mass"] = torch.tensor(d["m2"], dtype=torch.float64, device="cuda", requires_grad=True)
        s["U"] = d["U"].requires_grad_(True)
        s["spec"] = dict(dims=d["dims"], nc=case["nc"], p=d["p"], colors_dev=d["col"], ncolors=d["m"], seed=d["seed"],
                         nsamples=case["ns"], noise=case["noise"], dilute=case["dilute"], opts=s["opts"])
    return s


# ------------------------------------------------------------------ the calls


def _loss(T):
    return (T * (0.7 - 0.4j)).real


def run(s):
    ctx, kind = s["ctx"], s["kind"]
    if kind in ("trace", "batch"):
        res = ctx.trace_estimate(s["ops"], s["ps"], s["p"], s["opts"])
        if kind == "batch":  # all instances' results in one array each
            return {"T": np.array([r["T"] for r in res]), "per_sample": np.concatenate([r["per_sample"] for r in res]),
                    "tj": np.concatenate([r["tj"] for r in res])}
        return {"T": np.array([res[0]["T"]]), "per_sample": res[0]["per_sample"], "tj": res[0]["tj"]}
    if kind == "multi":
        res = ctx.trace_multi(s["ops"][0], s["ps"][0], list(range(s["p"][0] + 1)), s["opts"])
        return [{"T": np.array([r["T"]]), "per_sample": r["per_sample"], "tj": r["tj"]} for r in res]
    if kind == "deflated":
        r = ctx.trace_deflated(s["ops"][0], s["defl"], s["p"][0], s["ps"][0], s["opts"])
        return {"T": np.array([r["T"]]), "T_defl": np.array([r["T_defl"]]), "per_sample": r["per_sample"], "tj": r["tj"]}
    if kind == "grad":
        T, dm2, dU, dUb, st = ctx.trace_grad(s["ops"][0], s["ps"][0], s["p"][0], s["opts"])
        return {"T": np.array([T]), "dm2": np.array([dm2]), "dU": dU, "dUbar": dUb, "tj": st["tj"]}
    if kind == "autograd":
        s["mass"].grad = s["U"].grad = None
        T = dp.probed_trace(s["mass"], s["U"], **s["spec"])
        _loss(T).backward()
        return {"T": T.detach(), "dm2": s["mass"].grad, "dU": s["U"].grad}
    if kind == "apply":
        return {"y": ctx.apply(s["ops"][0], s["data"][0]["b"], s["inner"])}
    if kind == "noalloc":
        return {"x": ctx.solve_noalloc(s["ops"][0], s["data"][0]["b"], s["opts"])[0]}
    return {"x": ctx.solve_batch(s["ops"], [s["data"][0]["b"]], s["opts"])[0][0]}


# ------------------------------------------------------------------ 64-bit values


class _Op:
    """A on vectors [D0, D1, D2, D3, nc, R] in complex128 with plain torch."""

    def __init__(self, dims, nc, m2, U):
        self.diag = m2 + 8.0
        self.U = None if U is None else U.detach().reshape(4, *dims, nc, nc)
        self.shape = (*dims, nc)

    def __call__(self, v):
        out = self.diag * v
        for mu in range(4):
            up = torch.roll(v, -1, mu)
            if self.U is None:
                out = out - up - torch.roll(v, 1, mu)
                continue
            u = self.U[mu]
            nc = self.shape[-1]
            back = torch.zeros_like(v)
            for b in range(nc):
                out -= u[..., :, b, None] * up[..., b, None, :]
                back += u[..., b, :, None].conj() * v[..., b, None, :]
            out -= torch.roll(back, 1, mu)
        return out

    def solve(self, b):
        x, r, p = torch.zeros_like(b), b.clone(), b.clone()
        over = (0, 1, 2, 3, 4)
        bb = rr = (r.conj() * r).real.sum(over)
        for _ in range(400):
            q = self(p)
            a = rr / (p.conj() * q).real.sum(over).clamp_min(1e-300)
            x += a * p
            r -= a * q
            rn = (r.conj() * r).real.sum(over)
            p = r + (rn / rr.clamp_min(1e-300)) * p
            rr = rn
            if bool((rr <= 1e-30 * bb).all()):
                break
        r = b - self(x)  # one step of refinement on the true residual
        return x + (0 if float((r.abs().square().sum(over) / bb.clamp_min(1e-300)).max()) < 1e-28 else self.solve(r))


def _mix64(z):
    z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
    z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
    return z ^ (z >> np.uint64(31))


def _noise(seed, s, n, nc, kind):
    """z0(s, site, b), complex128 [n, nc], from the SplitMix64 counter hash."""
    ctr = np.uint64(s * n * nc) + np.arange(n * nc, dtype=np.uint64)
    h = _mix64(_mix64(np.array([seed], dtype=np.uint64)) ^ ctr)
    top, nxt = (h >> np.uint64(63)).astype(np.int64), ((h >> np.uint64(62)) & np.uint64(1)).astype(np.int64)
    if kind == "real_z2":
        z = 1.0 - 2.0 * top + 0j
    elif kind == "z2_complex":
        z = (1.0 - 2.0 * top) + 1j * (1.0 - 2.0 * nxt)
    else:
        z = np.array([1, 1j, -1, -1j])[2 * top + nxt]
    return torch.from_numpy(z.astype(np.complex128).reshape(n, nc)).cuda()


def _probes(case, d, j0, j1):
    """Probes j0 .. j1 - 1, [D0, D1, D2, D3, nc, R]."""
    n, nc = math.prod(d["dims"]), case["nc"]
    ndil = nc if case["dilute"] else 1
    v = torch.zeros((n, nc, j1 - j0), dtype=torch.complex128, device="cuda")
    z, zs = None, -1
    for j in range(j0, j1):
        s, c, a = j // (d["m"] * ndil), (j // ndil) % d["m"], j % ndil
        if s != zs:
            z, zs = _noise(d["seed"], s, n, nc, case["noise"]), s
        on = (d["col"] == c)[:, None] & ((torch.arange(nc, device="cuda") == a)[None] if case["dilute"] else True)
        v[:, :, j - j0] = torch.where(on, z, torch.zeros_like(z))
    return v.reshape(*d["dims"], nc, j1 - j0)


def _chunks(total, sites):
    w = max(1, min(total, 9_000_000 // sites))
    return [(j, min(total, j + w)) for j in range(0, total, w)]


def _estimates(case, d, disps, rhs=None):
    """{T, per_sample, tj} for every displacement; rhs(v): the right-hand sides of probes v."""
    A = _Op(d["dims"], case["nc"], d["m2"], d["U"])
    total = case["ns"] * d["m"] * (case["nc"] if case["dilute"] else 1)
    tj = [[] for _ in disps]
    for j0, j1 in _chunks(total, math.prod(d["dims"])):
        v = _probes(case, d, j0, j1)
        x = A.solve(v if rhs is None else rhs(v))
        for n, p in enumerate(disps):
            tj[n].append((v.conj() * torch.roll(x, -p, 0)).sum((0, 1, 2, 3, 4)).cpu().numpy())
    out = []
    for t in tj:
        t = np.concatenate(t)
        per = NORM[case["noise"]] * t.reshape(case["ns"], -1).sum(1)
        out.append({"T": np.array([per.mean()]), "per_sample": per, "tj": t})
    return out


def _gradient(case, d):
    A = _Op(d["dims"], case["nc"], d["m2"], d["U"])
    total = case["ns"] * d["m"] * (case["nc"] if case["dilute"] else 1)
    norm = NORM[case["noise"]] / case["ns"]
    n, nc, tj, dm2 = math.prod(d["dims"]), case["nc"], [], 0.0
    dU = torch.zeros((4, *d["dims"], nc, nc), dtype=torch.complex128, device="cuda")
    dUb = torch.zeros_like(dU)
    for j0, j1 in _chunks(total, n):
        v = _probes(case, d, j0, j1)
        x, lam = A.solve(v), A.solve(torch.roll(v, d["p"], 0))
        tj.append((v.conj() * torch.roll(x, -d["p"], 0)).sum((0, 1, 2, 3, 4)).cpu().numpy())
        dm2 = dm2 - norm * complex((lam.conj() * x).sum())
        for mu in range(4):
            xu, lu = torch.roll(x, -1, mu), torch.roll(lam, -1, mu)
            for a in range(nc):
                for b in range(nc):
                    dU[mu, ..., a, b] += norm * (lam[..., a, :].conj() * xu[..., b, :]).sum(-1)
                    dUb[mu, ..., a, b] += norm * (x[..., a, :] * lu[..., b, :].conj()).sum(-1)
    tj = np.concatenate(tj)
    return {"T": np.array([norm * tj.sum()]), "dm2": np.array([dm2]), "dU": dU.reshape(4, n, nc, nc),
            "dUbar": dUb.reshape(4, n, nc, nc), "tj": tj}


def exact(case, seed):
    kind = case["kind"]
    if kind == "deflated":
        return None  # needs the low eigenvectors of a large matrix
    data = _data(case, seed)
    if kind == "batch":
        res = [_estimates(case, d, [d["p"]])[0] for d in data]
        return {"T": np.concatenate([r["T"] for r in res]), "per_sample": np.concatenate([r["per_sample"] for r in res]),
                "tj": np.concatenate([r["tj"] for r in res])}
    d = data[0]
    if kind == "trace":
        return _estimates(case, d, [d["p"]])[0]
    if kind == "multi":
        return _estimates(case, d, list(range(d["p"] + 1)))
    if kind == "grad":
        return _gradient(case, d)
    if kind == "autograd":
        g = _gradient(case, d)
        w = 0.7 + 0.4j  # d Re(T (0.7 - 0.4i)) for PyTorch's convention
        return {"T": torch.tensor(complex(g["T"][0]), dtype=torch.complex128),
                "dm2": torch.tensor((np.conj(w) * g["dm2"][0]).real, dtype=torch.float64),
                "dU": np.conj(w) * g["dUbar"] + w * g["dU"].conj()}
    A = _Op(d["dims"], case["nc"], d["m2"], d["U"])
    out = torch.empty_like(d["b"])
    for j0, j1 in _chunks(case["nrhs"], math.prod(d["dims"])):
        v = d["b"][j0:j1].permute(1, 2, 0).reshape(*d["dims"], case["nc"], j1 - j0)
        y = A(v) if kind == "apply" else A.solve(v)
        out[j0:j1] = y.reshape(-1, case["nc"], j1 - j0).permute(2, 0, 1)
    return {"y" if kind == "apply" else "x": out}
