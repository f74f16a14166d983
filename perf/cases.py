"""The work that users of the library have it do, as cases that can be timed.

Kinds of case, each through the package's public entry points:

* ``product``  one operator product: ``apply_operator_noalloc`` (graph capture and serving
  loops, where the call may not allocate) or ``apply_operator_block`` (residual checks,
  kernel ridge predictions, a few columns at once);
* ``ridge``    kernel ridge regression: build the preconditioner, then solve for one
  right-hand side or a few (``solve`` / ``solve_batch``); explicit or basis-less;
* ``resolve``  a solve on a handle that the program keeps (more right-hand sides, later);
* ``dense``    a stored dense matrix: build and solve in float64, or in mixed precision;
* ``sweep``    many right-hand sides under several shifts on one joint-basis handle;
* ``serve``    a burst of independent requests through the continuous-batching server.

Sizes follow the workloads of ``workloads/`` and ``bench.py`` and the ranges between them.
"""
from __future__ import annotations

import math

import numpy as np
import torch

RBF, MATERN = 1, 2


def listed():
    return [
        # the smallest call: one float32-class product of a serving loop, bound by latency
        dict(name="product n=1000", kind="product", kernel=RBF, n=1000, d=4, prec="fp32", cols=1, entry="noalloc"),
        # a residual check in float64 (Matern-3/2 in three dimensions, an odd size)
        dict(name="product f64 n=20001", kind="product", kernel=MATERN, n=20001, d=3, prec="fp64", cols=1,
             entry="block"),
        # several columns at once at an ordinary size
        dict(name="product x8 n=16384", kind="product", kernel=RBF, n=16384, d=16, prec="fp32", cols=8, entry="block"),
        # the smallest and an ordinary, odd-sized request of the serving stream, each as one call pair
        dict(name="ridge n=1000", kind="ridge", n=1000, d=4, l=32, sketch="gaussian", basis="explicit", mu=1e-4,
             nrhs=1, tol=1e-6),
        dict(name="ridge x4 n=5793", kind="ridge", n=5793, d=8, l=182, sketch="gaussian", basis="explicit", mu=1e-4,
             nrhs=4, tol=1e-6),
        # the largest request of the stream
        dict(name="ridge x8 n=32768", kind="ridge", n=32768, d=16, l=1024, sketch="gaussian", basis="explicit",
             mu=1e-5, nrhs=8, tol=1e-6),
        # the headline: kernel ridge on 50,000 points of a 10-component mixture
        dict(name="ridge n=50000", kind="ridge", n=50000, d=16, l=500, sketch="srht", basis="explicit", mu=1e-4,
             nrhs=1, tol=1e-6),
        # its smaller shift on a kept handle: what each further right-hand side costs
        dict(name="resolve n=50000", kind="resolve", n=50000, d=16, l=500, sketch="srht", basis="explicit", mu=1e-6,
             nrhs=1, tol=1e-6),
        # the plain float64 method on a small stored matrix, iteration batches replayed as graphs
        dict(name="dense f64 n=2000", kind="dense", kernel=RBF, n=2000, d=8, l=100, prec="fp64", mu=1e-3, tol=1e-10),
        # the precision form at an ordinary size: float32 products, float64 refinement to 1e-10
        dict(name="dense mixed n=16384", kind="dense", kernel=MATERN, n=16384, d=3, l=512, prec="mixed", mu=1e-2,
             tol=1e-10),
        # a regularisation sweep: 64 right-hand sides under 4 shifts, refined to the same 1e-10
        dict(name="sweep 64x4 n=20000", kind="sweep", n=20000, d=16, l=400, sketch="srht", nrhs=64, shifts=4,
             tol=1e-10),
        # a burst of small and medium requests on the server
        dict(name="serve 12", kind="serve", requests=12, n_min=1000, n_max=8000, slots=8, tol=1e-6),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["product", "product", "ridge", "ridge", "ridge", "resolve", "dense", "sweep", "serve"])
    if kind == "product":
        entry = rng.choice(["noalloc", "block"])
        prec = rng.choice(["fp32", "fp32", "fp64"])
        n = _log_uniform(rng, 1000, 30000 if entry == "noalloc" else 50000)
        return dict(kind=kind, kernel=rng.choice([RBF, MATERN]), n=n, d=rng.choice([2, 3, 4, 5, 8, 11, 16]), prec=prec,
                    cols=1 if entry == "noalloc" else rng.choice([1, 2, 3, 4, 7, 8]), entry=entry)
    if kind in ("ridge", "resolve"):
        n = _log_uniform(rng, 1000, 50000)
        nrhs = rng.choice([1, 1, 2, 3, 5, 8]) if n <= 32768 else 1
        basis = "less" if kind == "ridge" and nrhs == 1 and rng.random() < 0.3 else "explicit"
        sketch = "colsample" if basis == "less" else rng.choice(["gaussian", "srht"])
        return dict(kind=kind, n=n, d=rng.choice([4, 8, 16]), l=min(1024, -(-n // rng.choice([32, 50, 100]))),
                    sketch=sketch, basis=basis, mu=10.0 ** -rng.uniform(3, 6), nrhs=nrhs, tol=1e-6)
    if kind == "dense":
        prec = rng.choice(["fp64", "mixed"])
        if prec == "fp64":
            n = _log_uniform(rng, 600, 4000)
            return dict(kind=kind, kernel=RBF, n=n, d=8, l=n // 20, prec=prec, mu=1e-3, tol=1e-10)
        n = _log_uniform(rng, 4000, 16384)
        return dict(kind=kind, kernel=MATERN, n=n, d=3, l=n // 32, prec=prec, mu=1e-2, tol=1e-10)
    if kind == "sweep":
        n = _log_uniform(rng, 5000, 20000)
        return dict(kind=kind, n=n, d=rng.choice([8, 16]), l=n // 50, sketch="srht", nrhs=rng.randint(12, 64),
                    shifts=rng.choice([3, 4]), tol=1e-10)
    return dict(kind=kind, requests=rng.randint(4, 12), n_min=1000, n_max=_log_uniform(rng, 2000, 8000), slots=8,
                tol=1e-6)


# ---------------------------------------------------------------- inputs

def _generator(seed, salt=0, device="cuda"):
    g = torch.Generator(device=device)
    g.manual_seed(1000003 * int(seed) + salt)
    return g


def _normal(g, *shape):
    return torch.randn(*shape, generator=g, device=g.device, dtype=torch.float64)


def _mixture(g, n, d, comps=10, mean_std=3.0):
    """(d, n) float32 points of an equal-weight mixture of unit-covariance Gaussians."""
    means = _normal(g, comps, d) * mean_std
    label = torch.randint(0, comps, (n,), generator=g, device=g.device)
    return (means[label] + _normal(g, n, d)).t().contiguous().float()


def _median_rule(pts):
    """1 / (2 sigma^2) with sigma the median distance among the first 2,000 points."""
    x = pts[:, :2000].double().t()
    r2 = torch.zeros(x.shape[0], x.shape[0], dtype=torch.float64, device=x.device)
    for k in range(x.shape[1]):
        r2 += (x[:, k, None] - x[None, :, k]) ** 2
    i, j = torch.triu_indices(x.shape[0], x.shape[0], 1, device=x.device)
    return float(np.float32(0.5 / float(torch.median(r2[i, j]))))


def _shifts(case):
    return [10.0 ** -(3 + k) for k in range(case["shifts"])]


def _problem(case, seed):
    """(kernel kind, points (d, n) float32, kernel constant, scale, right-hand sides (n, m)) of a case."""
    g = _generator(seed)
    n, d = case["n"], case["d"]
    if case["kind"] == "dense":
        if case["kernel"] == MATERN:
            pts = torch.rand(d, n, generator=g, device="cuda", dtype=torch.float64).float()
            return MATERN, pts, float(np.float32(math.sqrt(3.0) / 0.1)), 1.0, _normal(g, n, 1)
        return RBF, _normal(g, d, n).float(), 0.5, 1.0, _normal(g, n, 1)
    if case["kind"] == "product" and case["kernel"] == MATERN:
        pts = torch.rand(d, n, generator=g, device="cuda", dtype=torch.float64).float()
        return MATERN, pts, float(np.float32(math.sqrt(3.0) / 0.3)), 1.0 / n, _normal(g, n, case["cols"])
    pts = _mixture(g, n, d)
    m = case["cols"] if case["kind"] == "product" else case["nrhs"]
    return RBF, pts, _median_rule(pts), 1.0 / n, _normal(g, n, m)


def _request_size(case, rid):
    """(n, d): n spread evenly over its logarithm, in an order of its own."""
    t = ((rid * 5) % case["requests"] + 0.5) / case["requests"]
    return int(case["n_min"] * (case["n_max"] / case["n_min"]) ** t), (4, 8, 16)[rid % 3]


def _requests(case, seed):
    """Requests of the serving stream, all there at the start: host arrays, as a server receives them."""
    g = np.random.default_rng(1000003 * int(seed) + 5)
    out = []
    for rid in range(case["requests"]):
        n, d = _request_size(case, rid)
        pts = np.ascontiguousarray(g.standard_normal((n, d)).T.astype(np.float32))
        x = pts[:, :400].astype(np.float64).T
        r2 = ((x[:, None, :] - x[None, :, :]) ** 2).sum(-1)[np.triu_indices(x.shape[0], 1)]
        out.append(dict(kind=RBF, pts=pts, kconst=float(np.float32(0.5 / np.median(r2))), scale=1.0 / n,
                        mu=10.0 ** -(2 + 4 * ((rid * 7) % case["requests"]) / case["requests"]), l=-(-n // 32),
                        seed=1000 + rid, B=g.standard_normal((n, 1 + rid % 4)), t_arrival=0.0))
    return out


def prepare(case, seed):
    import paper_2509_19747_amd as rr

    if case["kind"] == "serve":
        return dict(case=case, requests=_requests(case, seed))
    kernel, pts, kconst, scale, B = _problem(case, seed)
    op = rr.kernel_operator(kernel, pts, kconst, scale)
    s = dict(case=case, op=op, B=B, b=B[:, 0].contiguous())
    if case["kind"] == "dense":
        s["op"] = rr.dense_operator(rr.kernel_to_dense(op, "fp64"))
    if case["kind"] == "product":
        s["y"] = torch.empty_like(s["b"])
    if case["kind"] == "resolve":
        s["handle"] = _build(rr, case, s)
    if case["kind"] == "sweep":
        s["handle"] = rr.build_precond(op, _shifts(case), l=case["l"], sketch=case["sketch"], seed=14, prec="fp32")
        s["B"] = B.repeat(1, case["shifts"])
        s["column shifts"] = [k for k in range(case["shifts"]) for _ in range(case["nrhs"])]
    return s


# ---------------------------------------------------------------- one pass

def _build(rr, case, s):
    return rr.build_precond(s["op"], [case["mu"]], l=case["l"], sketch=case["sketch"], seed=12, prec="fp32",
                            basis=case["basis"])


def _solve(case, s, handle):
    if case["nrhs"] == 1:
        return handle.solve(s["b"], tol=case["tol"], certify=False, check_every=8)[0]
    return handle.solve_batch(s["B"], [0] * case["nrhs"], tol=case["tol"], check_every=8)[0]


def run(state):
    import paper_2509_19747_amd as rr
    from paper_2509_19747_amd import binding

    s, case = state, state["case"]
    kind = case["kind"]
    if kind == "product":
        if case["entry"] == "noalloc":
            return binding.apply_operator_noalloc(s["op"], 1e-4, case["prec"], s["b"], y=s["y"])
        return rr.apply_operator_block(s["op"], 1e-4, case["prec"], s["B"])
    if kind == "ridge":
        return _solve(case, s, _build(rr, case, s))
    if kind == "resolve":
        return _solve(case, s, s["handle"])
    if kind == "dense":
        handle = rr.build_precond(s["op"], [case["mu"]], l=case["l"], sketch="gaussian", seed=11, prec=case["prec"])
        if case["prec"] == "fp64":
            return handle.solve(s["b"], tol=case["tol"], use_graph=True, check_every=16)[0]
        return handle.solve(s["b"], tol=case["tol"], certify=False, maxit=20000)[0]
    if kind == "sweep":
        return s["handle"].solve_batch(s["B"], s["column shifts"], tol=case["tol"], check_every=8)[0]
    results, _ = binding.serve(s["requests"], max_slots=case["slots"], build=dict(prec="fp32", sketch="gaussian"),
                               solve=dict(tol=case["tol"], certify=False))
    return [r["X"] for r in results]


# ---------------------------------------------------------------- minimum work

def work(case):
    """Inputs read once and outputs written once; the operations that any such pass does: every
    distinct kernel entry (2d + 1) and its use once in the sketch (2 n^2 l), the basis (4 n l^2) and one product
    for each right-hand side (how many more an iteration needs depends on the spectrum)."""
    if case["kind"] == "serve":
        b = f = 0.0
        for rid in range(case["requests"]):
            n, d = _request_size(case, rid)
            one = work(dict(kind="ridge", n=n, d=d, l=-(-n // 32), nrhs=1 + rid % 4))
            b, f = b + one["bytes"], f + one["flops"]
        return {"bytes": b, "flops": f}
    n, d = case["n"], case["d"]
    m = case["cols"] if case["kind"] == "product" else case.get("nrhs", 1) * case.get("shifts", 1)
    entries = (2 * d + 1) * n * (n + 1) / 2
    flops = entries + 2.0 * n * n * m
    nbytes = 4.0 * n * d + 16.0 * n * m
    if case["kind"] == "dense":
        nbytes = 8.0 * n * n + 16.0 * n
        flops = 2.0 * n * n
    if case["kind"] in ("ridge", "dense"):
        flops += 2.0 * n * n * case["l"] + 4.0 * n * case["l"] ** 2
    if case["kind"] in ("resolve", "sweep"):
        nbytes += 8.0 * n * case["l"] * (2 if case["kind"] == "sweep" else 1)
    return {"bytes": nbytes, "flops": flops}


# ---------------------------------------------------------------- 64 bits

class _Matrix:
    """scale * K(X, X) in float64, stored in blocks of rows."""

    ROWS = 2048

    def __init__(self, kernel, pts, kconst, scale):
        x = pts.double()
        n = x.shape[1]
        self.blocks = []
        for r0 in range(0, n, self.ROWS):
            xr = x[:, r0:r0 + self.ROWS]
            r2 = torch.zeros(xr.shape[1], n, dtype=torch.float64, device=x.device)
            for k in range(x.shape[0]):
                r2 += (xr[k][:, None] - x[k][None, :]) ** 2
            if kernel == RBF:
                self.blocks.append(torch.exp(r2.mul_(-kconst)).mul_(scale))
            else:
                r = r2.sqrt_().mul_(kconst)
                self.blocks.append((1.0 + r) * torch.exp(-r) * scale)

    def __matmul__(self, u):
        return torch.cat([b @ u for b in self.blocks])


def _cg(A, mu, B, iters=20000, tol=1e-14):
    """(A + mu I) X = B by conjugate gradients in float64, every column to tol or to rounding; mu: one shift a column."""
    X = torch.zeros_like(B)
    for _ in range(3):   # restarts from the true residual take the rounding of long recurrences out
        R = B - (A @ X + mu * X)
        P, rho = R.clone(), (R * R).sum(0)
        goal = tol * tol * (B * B).sum(0)
        for it in range(iters):
            if it % 25 == 0 and bool((rho <= goal).all()):
                break
            W = A @ P + mu * P
            live = rho > goal
            alpha = torch.where(live, rho / (P * W).sum(0), torch.zeros_like(rho))
            X += alpha * P
            R -= alpha * W
            new = (R * R).sum(0)
            P = R + torch.where(live, new / rho, torch.zeros_like(rho)) * P
            rho = torch.where(live, new, rho)
    return X


def exact(case, seed):
    if case["kind"] == "serve":
        out = []
        for r in _requests(case, seed):
            A = _Matrix(r["kind"], torch.from_numpy(r["pts"]).cuda(), r["kconst"], r["scale"])
            out.append(_cg(A, r["mu"], torch.from_numpy(r["B"]).cuda()).cpu().numpy())
        return out
    kernel, pts, kconst, scale, B = _problem(case, seed)
    A = _Matrix(kernel, pts, kconst, scale)
    if case["kind"] == "product":
        Y = A @ B + 1e-4 * B
        return Y[:, 0].contiguous() if case["entry"] == "noalloc" else Y
    if case["kind"] == "sweep":
        mu = torch.tensor(_shifts(case), dtype=torch.float64, device="cuda").repeat_interleave(case["nrhs"])
        return _cg(A, mu, B.repeat(1, case["shifts"]))
    X = _cg(A, case["mu"], B)
    return X[:, 0].contiguous() if case["kind"] == "dense" or case["nrhs"] == 1 else X
