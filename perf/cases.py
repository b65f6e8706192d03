"""Workloads that stand for the use of this library, for timing it.

Each case is one call of a public entry point (or the short sequence a program
makes of it) at sizes from the repository's own configurations, tests and
benchmark.  ``listed()`` gives fixed cases, ``draw(rng)`` further ones of the
same ranges; ``prepare`` builds what a program holds before the call (the
handle of its problem, factor, dual, model), ``run`` makes one pass,
``work`` counts the bytes and operations one pass cannot do without and
``exact`` gives the outputs in 64-bit arithmetic of plain torch.

Graphs are built on the GPU (seeded), since the largest one has 8e7 entries.
"""

import math

import numpy as np
import torch

import gen
import paper_2505_15775_amd as almbm
from paper_2505_15775_amd import _lib, warmstart

DEV = "cuda:0"
VBYTES = {"f64": 8, "f32": 4, "bf16": 4}  # stored cost value
SBYTES = {"f64": 8, "f32": 4, "bf16": 2}  # stored factor entry


# ----------------------------------------------------------------- the cases


def listed():
    return [
        # The smallest call: one objective and gradient at the plain FP64 workload (n = 2000, degree 10,
        # unit weights, r = 8), as a program with its own outer loop makes it.  Bound by launches.
        dict(name="objgrad_er2000_f64", kind="objgrad", graph="er", n=2000, deg=10.0, weights="unit", r=8, prec="f64"),
        # The same call on a power-law graph (R-MAT), where a few rows hold most entries.
        dict(name="objgrad_rmat18_f64", kind="objgrad", graph="rmat", n=1 << 18, deg=16.0, weights="gauss", r=16,
             prec="f64"),
        # The headline: gradient-descent steps of the subproblem at n = 1e7, BF16 factor.
        dict(name="gd_er1e7_bf16", kind="inner", graph="er", n=10_000_000, deg=8.0, weights="gauss", r=16,
             prec="bf16", solver="gd", steps=20, sigma=16.0),
        # Gradient-descent steps on the 1000 x 1000 torus with +-1 weights in FP32: mesh-like locality.
        dict(name="gd_torus1e6_f32", kind="inner", graph="torus", n=1_000_000, deg=4.0, weights="pm1", r=16,
             prec="f32", solver="gd", steps=30, sigma=1.0),
        # L-BFGS steps (memory 3) in FP64 at the size of the largest instance of the uneven batch.
        dict(name="lbfgs_er193176_f64", kind="inner", graph="er", n=193_176, deg=18.0, weights="pm1", r=16,
             prec="f64", solver="lbfgs", steps=16, sigma=16.0),
        # The eigenvalue check of every outer iteration: Lanczos passes of up to 60 columns, restarted until the
        # residual meets the tolerance of a solve to 1e-4 relative KKT.
        dict(name="lanczos_er1e6", kind="lanczos", graph="er", n=1_000_000, deg=8.0, weights="gauss", kmax=60,
             prec="f64"),
        # Lovasz theta at its configured size (n = 1e5, 1e6 edges, r = 32, FP32): sampled products on edges.
        dict(name="objgrad_lovasz1e5_f32", kind="lovasz", n=100_000, deg=20.0, r=32, prec="f32"),
        # Matrix completion (Table 2, n = 2e4, rank 3: long rows, narrow odd rank), gradient-descent steps.
        dict(name="gd_completion2e4_f64", kind="completion", n=20_000, r=3, prec="f64", steps=30, sigma=0.03),
        # Learned warm start, inference: features, dual and pooled features of a graph.
        dict(name="warm_predict_er1e6", kind="predict", graph="er", n=1_000_000, deg=8.0, weights="gauss"),
        # Learned warm start, training: loss and gradient of one minibatch of fit().
        dict(name="warm_train_262144", kind="train", n=1 << 18, h=32),
        # A whole batched solve of uneven instances (the batch recipe), stopped after two outer iterations.
        dict(name="batch24_f64", kind="batch", n=40_000, count=24, prec="f64", r=16, outer=2, inner=40, sigma=16.0),
        # A whole solve of the plain FP64 workload, stopped after three outer iterations.
        dict(name="solve_er2000_f64", kind="solve", graph="er", n=2000, deg=10.0, weights="unit", r=8, prec="f64",
             outer=3, inner=200, sigma=1.0),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["objgrad", "objgrad", "inner", "inner", "lanczos", "lovasz", "completion", "predict", "train",
                       "batch", "solve"])
    prec = rng.choice(["f64", "f32", "bf16"])
    weights = rng.choice(["unit", "pm1", "gauss"])
    graph = rng.choice(["er", "er", "torus", "rmat"])
    rank = rng.choice([4, 8, 16, 32, 64, rng.randint(3, 40)])
    deg = round(rng.uniform(4.0, 32.0), 2)
    if kind in ("objgrad", "inner"):
        n = _log_int(rng, 1_000, 1_000_000)
        if graph == "rmat":
            n, deg = 1 << rng.randint(11, 18), 16.0
        elif graph == "torus":
            a = max(3, int(math.sqrt(n)))
            n, deg = a * a, 4.0
        c = dict(kind=kind, graph=graph, n=n, deg=deg, weights=weights, r=rank, prec=prec)
        if kind == "inner":
            c.update(solver=rng.choice(["gd", "lbfgs"]), steps=rng.randint(8, 24), sigma=rng.choice([1.0, 16.0]))
            if c["solver"] == "lbfgs":  # a quasi-Newton path repeats rounding only over a few steps
                c["steps"] = rng.randint(4, 8)
        return c
    if kind == "lanczos":
        if graph == "rmat":
            n, deg = 1 << rng.randint(11, 18), 16.0
        else:
            graph, n = "er", _log_int(rng, 2_000, 700_000)
        return dict(kind=kind, graph=graph, n=n, deg=deg, weights="gauss", kmax=rng.randint(80, 120), prec="f64")
    if kind == "lovasz":
        return dict(kind=kind, n=_log_int(rng, 500, 100_000), deg=round(rng.uniform(8.0, 20.0), 2), r=rank,
                    prec=rng.choice(["f64", "f32"]))
    if kind == "completion":
        return dict(kind=kind, n=2 * _log_int(rng, 500, 10_000), r=rng.choice([3, 5]), prec="f64",
                    steps=rng.randint(8, 30), sigma=0.03)
    if kind == "predict":
        n, deg = _log_int(rng, 10_000, 1_000_000), round(rng.uniform(4.0, 16.0), 2)
        if graph == "torus":
            n, deg = math.isqrt(n) ** 2, 4.0
        return dict(kind=kind, graph="torus" if graph == "torus" else "er", n=n, deg=deg, weights=weights)
    if kind == "train":
        return dict(kind=kind, n=_log_int(rng, 5_000, 1 << 18), h=rng.choice([16, 32, 64]))
    if kind == "batch":
        return dict(kind=kind, n=_log_int(rng, 2_000, 40_000), count=rng.randint(4, 24), prec="f64", r=16, outer=2,
                    inner=rng.randint(10, 40), sigma=16.0)
    return dict(kind="solve", graph="er", n=_log_int(rng, 1_000, 50_000), deg=deg, weights=weights,
                r=rng.choice([4, 8, 16]), prec="f64", outer=2, inner=rng.randint(20, 100), sigma=16.0)


# ----------------------------------------------------------------- inputs


def _gen(seed, salt=0):
    return torch.Generator(device=DEV).manual_seed(int(seed) * 7919 + salt)


def _edges(case, seed):
    """(n, lower end, upper end, weight) of the case's graph, edges sorted by (i, j)."""
    n, g = int(case["n"]), _gen(seed)
    if case["graph"] == "torus":
        a = math.isqrt(n)
        v = torch.arange(n, device=DEV).view(a, a)
        i = torch.cat([v.reshape(-1), v.reshape(-1)])
        j = torch.cat([v.roll(-1, 0).reshape(-1), v.roll(-1, 1).reshape(-1)])
    elif case["graph"] == "rmat":
        m, bits = int(n * case["deg"] / 2), n.bit_length() - 1
        i = torch.zeros(m, dtype=torch.int64, device=DEV)
        j = torch.zeros(m, dtype=torch.int64, device=DEV)
        for bit in range(bits):  # quadrant probabilities 0.57, 0.19, 0.19, 0.05
            u = torch.rand(m, device=DEV, generator=g)
            i |= (u >= 0.76).long() << bit
            j |= (((u >= 0.57) & (u < 0.76)) | (u >= 0.95)).long() << bit
    else:
        m = min(int(n * case["deg"] / 2), n * (n - 1) // 4)
        k = int(m * 1.05) + 64 + 2 * m * m // (n * n)
        i = torch.randint(0, n, (k,), device=DEV, generator=g)
        j = torch.randint(0, n, (k,), device=DEV, generator=g)
    keep = i != j
    lo, hi = torch.minimum(i, j)[keep], torch.maximum(i, j)[keep]
    del i, j, keep
    key = torch.unique(lo * n + hi)
    if case["graph"] == "er" and key.numel() > m:
        drop = torch.randperm(key.numel(), device=DEV, generator=g)[: key.numel() - m]
        keep = torch.ones(key.numel(), dtype=torch.bool, device=DEV)
        keep[drop] = False
        key = key[keep]
    lo, hi = key // n, key % n
    if case["weights"] == "unit":
        w = torch.ones(key.numel(), dtype=torch.float64, device=DEV)
    elif case["weights"] == "pm1":
        w = torch.randint(0, 2, (key.numel(),), device=DEV, generator=g).double() * 2 - 1
    else:
        # multiples of 2^-20, so that sums of weights do not depend on their order
        w = (torch.randn(key.numel(), dtype=torch.float64, device=DEV, generator=g) * 2.0 ** 20).round() / 2.0 ** 20
    return n, lo, hi, w


def _cost(case, seed):
    """The MaxCut cost C = -L/4 as CSR (off-diagonal) and diagonal, on the GPU."""
    n, lo, hi, w = _edges(case, seed)
    row, col, val = torch.cat([lo, hi]), torch.cat([hi, lo]), torch.cat([w, w]) * 0.25
    dg = torch.zeros(n, dtype=torch.float64, device=DEV).index_add_(0, row, -val)
    rp = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    rp[1:] = torch.bincount(row, minlength=n).cumsum(0)
    key = row * n + col
    del lo, hi, w, row, col
    key, order = torch.sort(key)
    return n, rp.int(), (key % n).int(), val[order].contiguous(), dg


def _maxcut(case, seed, r_max, kmax=0, lbfgs=0):
    """The handle of Problem.maxcut for a cost that is on the GPU already."""
    n, rp, ci, cv, dg = _cost(case, seed)
    b = torch.ones(n, dtype=torch.float64, device=DEV)
    arrays = dict(row_ptr=rp, col_idx=ci, val=cv, diag=dg, b=b)
    kw = dict(n=n, nnz=ci.numel(), row_ptr=rp.data_ptr(), col_idx=ci.data_ptr(), val=cv.data_ptr(), ell_width=0,
              diag=dg.data_ptr(), j_coef=0.0, cons_kind=_lib.CONS_DIAG, m=n, b=b.data_ptr(), trace_coef=0.0,
              n_edges=0, edge_i=0, edge_j=0, precision=_lib.PRECISIONS[case.get("prec", "f64")], r_max=r_max,
              lanczos_kmax=kmax, validate=0, rank_block_max=0, lbfgs_memory_max=lbfgs, hub_min_degree=0)
    return almbm.Problem(kw, arrays, case.get("prec", "f64"), DEV), arrays


def _factor(n, r, seed, dtype, noise=0.0):
    """Rows N(0,1) scaled to unit length (the solves' start), with `noise` on top for a point of the path."""
    g = _gen(seed, 1)
    R = torch.randn((n, r), dtype=torch.float32, device=DEV, generator=g)
    R /= R.norm(dim=1, keepdim=True).clamp_min(1e-30)
    if noise:
        R += noise * torch.randn((n, r), dtype=torch.float32, device=DEV, generator=g)
    return R.to(dtype).contiguous()


def _dual(arrays, n, seed):
    """A dual of the size solves meet: most of the way to the Gershgorin bound d_i - sum_j |S_ij|, with noise."""
    rows = torch.repeat_interleave(torch.arange(n, device=DEV), (arrays["row_ptr"][1:] - arrays["row_ptr"][:-1]).long())
    a = torch.zeros(n, dtype=torch.float64, device=DEV).index_add_(0, rows, arrays["val"].abs())
    u = torch.rand(n, dtype=torch.float64, device=DEV, generator=_gen(seed, 2))
    return arrays["diag"] - a * (0.6 + 0.4 * u)


def _lanczos_tol(arrays):
    """Residual a solve to 1e-4 relative KKT asks for: 0.1 eps (1 + ||C||_F)."""
    return 1e-5 * (1.0 + math.sqrt(_dot(arrays["val"], arrays["val"]) + _dot(arrays["diag"], arrays["diag"])))


def _lovasz(case, seed):
    n, lo, hi, _ = _edges(dict(case, graph="er", weights="unit"), seed)
    p = almbm.Problem.lovasz(n, lo.cpu().numpy(), hi.cpu().numpy(), precision=case["prec"], r_max=case["r"],
                             lanczos_kmax=0, device=DEV, validate=False)
    R = _factor(n, case["r"], seed, p.dtype, 0.1)
    R /= R.norm()
    y = torch.randn(p.m, dtype=torch.float64, device=DEV, generator=_gen(seed, 2))
    y[0] = -float(n) / 50
    return p, lo, hi, R, y


def _completion(case, seed):
    """Observed entries of a random rank-r matrix (the sample count of the completion recipe)."""
    n, r = int(case["n"]), int(case["r"])
    n1, n2 = n // 2, n - n // 2
    g = _gen(seed)
    U = torch.randn((n1, r), dtype=torch.float64, device=DEV, generator=g)
    V = torch.randn((n2, r), dtype=torch.float64, device=DEV, generator=g)
    m = gen.sample_count(n1, n2, r)
    if 2 * m > n1 * n2:
        key = torch.randperm(n1 * n2, device=DEV, generator=g)[:m].sort().values
    else:
        key = torch.unique(torch.randint(0, n1 * n2, (m + m // 3 + 16,), device=DEV, generator=g))
        key = key[torch.randperm(key.numel(), device=DEV, generator=g)[:m].sort().values]
    rows, cols = key // n2, key % n2
    vals = (U[rows] * V[cols]).sum(1)
    R = torch.cat([U, V]) + 0.3 * torch.randn((n, r), dtype=torch.float64, device=DEV, generator=g)
    y = 0.05 * torch.randn(m + 1, dtype=torch.float64, device=DEV, generator=g)
    y[0] = 0.0
    return n1, n2, rows, cols, vals, R.contiguous(), y


def _batch_graphs(case, seed):
    """Instances of the uneven batch recipe, sizes log-uniform in [1e3, n] (the same for every seed)."""
    rng = np.random.default_rng(int(case["n"]) + int(case["count"]))
    for q in range(int(case["count"])):
        n = int(round(math.exp(rng.uniform(math.log(1e3), math.log(case["n"])))))
        yield dict(graph="er", n=n, deg=float(rng.uniform(4.0, 32.0)), weights="pm1", prec=case["prec"]), q, int(
            rng.choice([8, 16]))


def prepare(case, seed):
    kind, s = case["kind"], {"case": case}
    if kind == "objgrad":
        p, a = _maxcut(case, seed, case["r"])
        s.update(p=p, R=_factor(p.n, case["r"], seed, p.dtype, 0.1), y=_dual(a, p.n, seed))
    elif kind == "inner":
        p, a = _maxcut(case, seed, case["r"], lbfgs=3 if case["solver"] == "lbfgs" else 0)
        s.update(p=p, R=_factor(p.n, case["r"], seed, p.dtype), y=_dual(a, p.n, seed))
    elif kind == "lanczos":
        p, a = _maxcut(case, seed, 4, kmax=case["kmax"])
        s.update(p=p, y=_dual(a, p.n, seed), tol=_lanczos_tol(a))
    elif kind == "lovasz":
        p, _, _, R, y = _lovasz(case, seed)
        s.update(p=p, R=R, y=y)
    elif kind == "completion":
        n1, n2, rows, cols, vals, R, y = _completion(case, seed)
        p = almbm.Problem.matrix_completion(n1, n2, rows.cpu().numpy(), cols.cpu().numpy(), vals.cpu().numpy(),
                                            precision=case["prec"], r_max=8, lanczos_kmax=0, device=DEV,
                                            validate=False)
        s.update(p=p, R=R, y=y)
    elif kind == "predict":
        p, _ = _maxcut(case, seed, 4)
        s.update(p=p, model=warmstart.WarmStartModel.load(device=DEV))
    elif kind == "train":
        X, T = _train_set(case, seed)
        model = warmstart.WarmStartModel(h=case["h"], device=DEV, seed=int(seed) % 1000)
        model.mu, model.inv_sd = X.mean(dim=0).contiguous(), (1.0 / X.std(dim=0)).contiguous()
        s.update(model=model, X=X, T=T)
    elif kind == "batch":
        probs, factors = [], []
        for c, q, r in _batch_graphs(case, seed):
            p, _ = _maxcut(c, int(seed) * 64 + q, 32, kmax=40)
            probs.append(p)
            factors.append(_factor(p.n, r, int(seed) * 64 + q, p.dtype))
        s.update(batch=almbm.Batch(probs, rank_stride=32), factors=factors)
        for p in probs:
            p.close()
    else:
        p, _ = _maxcut(case, seed, 48, kmax=60)
        s.update(p=p, R=_factor(p.n, case["r"], seed, p.dtype))
    return s


def _train_set(case, seed):
    """Feature rows with the spreads the feature kernel gives (log degree, weighted sums, bound) and dual targets."""
    g = _gen(seed)
    z = torch.randn((int(case["n"]), 8), device=DEV, generator=g)
    scale = torch.tensor([0.3, 0.7, 0.7, 0.7, 1.0, 0.1, 0.2, 0.3], device=DEV)
    shift = torch.tensor([2.2, 1.6, 0.0, 0.0, -1.6, 2.2, 2.6, 1.7], device=DEV)
    X = (z * scale + shift).contiguous()
    T = (0.8 * X[:, 4] + 0.1 * X[:, 0] * X[:, 7] + 0.05 * torch.randn(X.shape[0], device=DEV, generator=g)).contiguous()
    return X, T


# ----------------------------------------------------------------- one pass

_RESULT = ("outer", "inner_total", "rank", "expansions", "pobj", "dobj", "pinf")


def run(s):
    c = s["case"]
    kind = c["kind"]
    if kind in ("objgrad", "lovasz"):
        f, G, Av = s["p"].objective_grad(s["R"], s["y"], 1.3)
        return {"f": f, "G": G, "Av": Av}
    if kind in ("inner", "completion"):
        R = s["R"].clone()
        opts = {}
        if c.get("solver") == "lbfgs":
            opts = dict(inner_solver=_lib.INNER_LBFGS, lbfgs_memory=3)
        steps, flag, f = s["p"].inner_solve(R, s["y"], 0.0, c["steps"], sigma=c["sigma"], **opts)
        return {"R": R, "f": f, "steps": steps, "flag": flag}
    if kind == "lanczos":
        theta, v, resid, iters = s["p"].lanczos_min_eig(s["y"], max_iter=c["kmax"], tol=s["tol"], seed=1)
        return {"theta": theta, "v": v, "resid": resid, "iters": iters}
    if kind == "predict":
        F = warmstart.features(s["p"])
        y0 = s["model"].predict_y0(s["p"], F)
        pool = warmstart.pooled(F)
        return {"F": F, "y0": y0, "pool": pool, "r0": s["model"].predict_r0(pool, s["p"].n)}
    if kind == "train":
        loss, grad = s["model"].loss_grad(s["X"], s["T"])
        return {"loss": loss, "grad": grad}
    if kind == "batch":
        _, st, res, R, ranks, y = s["batch"].solve(s["factors"], eps_kkt=1e-6, sigma=c["sigma"], max_outer=c["outer"],
                                                   max_inner=c["inner"], lanczos_restarts=0)
        return {"R": R, "y": y, "ranks": np.array(ranks), "status": np.array(st),
                "results": np.array([[float(r[k]) for k in _RESULT] for r in res])}
    st, res, R, y = s["p"].solve(s["R"], eps_kkt=1e-6, sigma=c["sigma"], max_outer=c["outer"], max_inner=c["inner"],
                                 lanczos_restarts=0)
    return {"R": R, "y": y, "status": st, "results": np.array([float(res[k]) for k in _RESULT])}


# ----------------------------------------------------------------- what a pass cannot do without


def _step_work(n, nnz, r, prec, m):
    """One gradient evaluation: the cost once, the factor read and the gradient (or new factor) written."""
    return (4 * (n + 1) + nnz * (4 + VBYTES[prec]) + n * VBYTES[prec] + 2 * n * r * SBYTES[prec] + 3 * m * 8,
            2.0 * nnz * r + 12.0 * n * r)


def _lanczos_work(n, nnz, kmax, passes):
    """Per step the product and, for the two projections, one read of the basis each."""
    by = sum(4 * (n + 1) + 12 * nnz + 4 * 8 * n + 2 * 8 * n * (j + 1) for j in range(kmax))
    return passes * by, passes * sum(2.0 * nnz + 8.0 * n * (j + 1) for j in range(kmax))


def work(case):
    kind, n = case["kind"], int(case["n"])
    r, prec = int(case.get("r", 0)), case.get("prec", "f64")
    nnz = int(n * case.get("deg", 0.0))
    if kind in ("objgrad", "inner", "lovasz"):
        b, f = _step_work(n, nnz, r, prec, n if kind != "lovasz" else nnz // 2)
        k = case.get("steps", 1)
        if kind == "inner":  # each step needs a gradient and the product of its direction
            f *= 2
    elif kind == "completion":
        m = gen.sample_count(n // 2, n - n // 2, r)
        k, b, f = case["steps"], 2 * n * r * 8 + m * (4 + 16), 16.0 * m * r
    elif kind == "lanczos":
        k = 1
        b, f = _lanczos_work(n, nnz, case["kmax"], 1)
    elif kind == "predict":
        k, b, f = 1, 4 * (n + 1) + 12 * nnz + 8 * n + 40 * n, n * 2.0 * (8 * 32 + 32 * 32 + 32)
    elif kind == "train":
        h = case["h"]
        k, b, f = 1, n * 36, n * 6.0 * (8 * h + h * h + h)
    elif kind == "batch":
        k, b, f = 1, 0.0, 0.0
        for c, _, rq in _batch_graphs(case, 0):
            nz = int(c["n"] * c["deg"])
            sb, sf = _step_work(c["n"], nz, rq, prec, c["n"])
            lb, lf = _lanczos_work(c["n"], nz, 40, 2)
            b += case["outer"] * (case["inner"] * sb + lb)
            f += case["outer"] * (case["inner"] * 2 * sf + lf)
    else:
        sb, sf = _step_work(n, nnz, r, prec, n)
        lb, lf = _lanczos_work(n, nnz, 60, 2)
        k, b, f = case["outer"], case["inner"] * sb + lb, case["inner"] * 2 * sf + lf
    return {"bytes": float(k * b), "flops": float(k * f)}


# ----------------------------------------------------------------- 64-bit values


class _Cost:
    """C = S + Diag(d) in FP64 on the GPU, applied to the columns of X a few at a time."""

    def __init__(self, case, seed):
        self.n, rp, ci, self.cv, self.dg = _cost(case, seed)
        self.S = torch.sparse_csr_tensor(rp, ci, self.cv, (self.n, self.n))
        self.arrays = dict(row_ptr=rp, col_idx=ci, val=self.cv, diag=self.dg)

    def __call__(self, X):
        return torch.sparse.mm(self.S, X) + self.dg[:, None] * X


def _argmin_quartic(k):
    """Smallest minimiser over t >= 0 of sum_i k[i] t^i (0 if there is none)."""
    t = np.roots([4 * k[4], 3 * k[3], 2 * k[2], k[1]])
    t = [0.0] + sorted(float(x.real) for x in t if abs(x.imag) < 1e-9 * (1 + abs(x.real)) and x.real > 0)
    return min(t, key=lambda x: sum(c * x ** i for i, c in enumerate(k)))


def _dot(a, b):
    return float((a * b).sum())


def _exact_steps(cost, amap, b, y, sigma, R, steps, memory, adj):
    """`steps` steps of gradient descent (memory 0) or L-BFGS with the exact line search; (R, objective at R)."""
    pairs, E, G_old, t = [], None, None, 0.0
    for k in range(steps + 1):
        P, a = cost(R), amap(R, R)
        e = a - b
        w = y - sigma * e
        f = _dot(R, P) + _dot(y, b - a) + 0.5 * sigma * _dot(e, e)
        if k == steps:
            return R, f
        G = 2 * (P - adj(w, R))
        if E is not None and memory:
            s_k, y_k = -t * E, G - G_old
            if t <= 0:
                pairs = []
            elif _dot(s_k, y_k) > 1e-12 * float(s_k.norm() * y_k.norm()):
                pairs = (pairs + [(s_k, y_k)])[-memory:]
        q, al = G, []
        for s_i, y_i in reversed(pairs):
            al.append(_dot(s_i, q) / _dot(s_i, y_i))
            q = q - al[-1] * y_i
        if pairs:
            q = q * (_dot(*pairs[-1]) / _dot(pairs[-1][1], pairs[-1][1]))
        for (s_i, y_i), a_i in zip(pairs, reversed(al)):
            q = q + (a_i - _dot(y_i, q) / _dot(s_i, y_i)) * s_i
        if pairs and _dot(q, G) <= 0:
            pairs, q = [], G
        E, G_old = q, G
        a1, a2 = 2 * amap(R, E), amap(E, E)
        t = _argmin_quartic([f, -2 * _dot(E, P) + _dot(y, a1) - sigma * _dot(e, a1),
                             _dot(E, cost(E)) - _dot(y, a2) + 0.5 * sigma * (_dot(a1, a1) + 2 * _dot(e, a2)),
                             -sigma * _dot(a1, a2), 0.5 * sigma * _dot(a2, a2)])
        R = R - t * E


def _exact_lanczos(cost, y, kmax, tol):
    """Smallest Ritz value, its residual and the columns built, by Krylov spaces of at most kmax columns, the first
    from the counter-based random vector, up to three more from the Ritz vector of the one before while the residual
    exceeds tol; a space ends where the residual estimate, looked at every 8 columns (4 up to n = 4096), meets tol."""
    n = y.numel()

    def z(x):
        return cost(x[:, None])[:, 0] - y * x

    m64 = (1 << 64) - 1

    def signed(v):
        v &= m64
        return v - (1 << 64) if v >> 63 else v

    def shift(v, b):  # logical right shift
        return (v >> b) & ((1 << (64 - b)) - 1)

    c1, c2 = signed(0xbf58476d1ce4e5b9), signed(0x94d049bb133111eb)
    u = torch.arange(1, n + 1, device=DEV) * c1 + signed(0x9e3779b97f4a7c15)
    u = (u ^ shift(u, 30)) * c1
    u = (u ^ shift(u, 27)) * c2
    u = u ^ shift(u, 31)
    v = shift(u, 11).double() * (2.0 / 2 ** 53) - 1.0
    kmax, every, total = min(kmax, n), 4 if n <= 4096 else 8, 0
    for _ in range(4):
        Q = torch.zeros((kmax, n), dtype=torch.float64, device=DEV)
        Q[0] = v / v.norm()
        T = torch.zeros((kmax, kmax), dtype=torch.float64, device=DEV)
        for j in range(kmax):
            x = z(Q[j])
            for _ in range(2):
                h = (Q[: j + 1] * x).sum(1)
                x = x - (Q[: j + 1] * h[:, None]).sum(0)
                T[j, j] += h[j]
            m, beta = j + 1, float(x.norm())
            if m % every == 0 or m == kmax:
                lam, U = torch.linalg.eigh(T[:m, :m].cpu())
                if beta * abs(float(U[-1, 0])) <= tol or m == kmax:
                    break
            T[j, j + 1] = T[j + 1, j] = beta
            Q[j + 1] = x / beta
        total += m
        v = (Q[:m] * U[:, 0].to(DEV)[:, None]).sum(0)
        v = v / v.norm()
        resid = float((z(v) - lam[0].item() * v).norm())
        if resid <= tol:
            break
    return float(lam[0]), resid, total


def exact(case, seed):
    kind = case["kind"]
    if kind in ("objgrad", "inner"):
        dt = almbm.TORCH_DTYPES[case["prec"]]
        C = _Cost(case, seed)
        y = _dual(C.arrays, C.n, seed)
        R = _factor(C.n, case["r"], seed, dt, 0.1 if kind == "objgrad" else 0.0).double()
        if kind == "inner":
            R, f = _exact_steps(C, lambda A, B: (A * B).sum(1), 1.0, y, case["sigma"], R, case["steps"],
                                3 if case["solver"] == "lbfgs" else 0, lambda w, X: w[:, None] * X)
            return {"R": R, "f": f, "steps": None, "flag": None}
        P, a = C(R), (R * R).sum(1)
        e = a - 1.0
        f = _dot(R, P) - _dot(y, e) + 0.65 * _dot(e, e)
        return {"f": torch.tensor([f], dtype=torch.float64), "G": 2 * (P - (y - 1.3 * e)[:, None] * R), "Av": a}
    if kind == "lanczos":
        C = _Cost(case, seed)
        theta, resid, iters = _exact_lanczos(C, _dual(C.arrays, C.n, seed), case["kmax"], _lanczos_tol(C.arrays))
        return {"theta": theta, "v": None, "resid": resid, "iters": iters}  # v has no sign of its own
    if kind == "lovasz":
        p, lo, hi, R, y = _lovasz(case, seed)
        R = R.double()
        a = torch.cat([(R * R).sum().view(1), (R[lo] * R[hi]).sum(1)])
        e = a.clone()
        e[0] -= 1.0
        w = y - 1.3 * e
        cs = R.sum(0)
        f = -_dot(cs, cs) - _dot(y, e) + 0.65 * _dot(e, e)
        ad = w[0] * R
        ad = ad.index_add(0, lo, 0.5 * w[1:, None] * R[hi]).index_add(0, hi, 0.5 * w[1:, None] * R[lo])
        return {"f": torch.tensor([f], dtype=torch.float64), "G": 2 * (-cs[None, :] - ad), "Av": a}
    if kind == "completion":
        n1, n2, rows, cols, vals, R, y = _completion(case, seed)
        j = n1 + cols
        b = torch.cat([torch.zeros(1, dtype=torch.float64, device=DEV), vals])
        zero = torch.zeros(1, dtype=torch.float64, device=DEV)

        def amap(A, B):
            return torch.cat([zero, 0.5 * ((A[rows] * B[j]).sum(1) + (B[rows] * A[j]).sum(1))])

        def adj(w, X):
            u = 0.5 * w[1:, None]
            return torch.zeros_like(X).index_add(0, rows, u * X[j]).index_add(0, j, u * X[rows])

        R, f = _exact_steps(lambda X: 0.5 * X, amap, b, y, case["sigma"], R, case["steps"], 0, adj)
        return {"R": R, "f": f, "steps": None, "flag": None}
    if kind == "predict":
        return _exact_predict(case, seed)
    if kind == "train":
        X, T = _train_set(case, seed)
        model = warmstart.WarmStartModel(h=case["h"], device=DEV, seed=int(seed) % 1000)
        mu, isd = X.mean(dim=0).double(), (1.0 / X.std(dim=0)).double()
        par = model.params.double().requires_grad_()
        loss = ((_mlp(par, 8, case["h"], (X.double() - mu) * isd) - T.double()) ** 2).mean()
        loss.backward()
        return {"loss": loss.detach().view(1), "grad": par.grad}
    return None  # whole solves: their path is compared with itself


def _mlp(par, nin, h, x):
    sizes, o, out = (nin * h, h, h * h, h, h, 1), 0, []
    for k in sizes:
        out.append(par[o:o + k])
        o += k
    W1, b1, W2, b2, W3, b3 = out
    z = torch.relu(x @ W1.view(nin, h) + b1)
    z = torch.relu(z @ W2.view(h, h) + b2)
    return z @ W3 + b3


def _exact_predict(case, seed):
    n, rp, ci, cv, dg = _cost(case, seed)
    deg = (rp[1:] - rp[:-1]).long()
    rows = torch.repeat_interleave(torch.arange(n, device=DEV), deg)

    def rowsum(v):
        return torch.zeros(n, dtype=torch.float64, device=DEV).index_add_(0, rows, v)

    nz = (cv != 0).double()
    ld, sa = torch.log1p(rowsum(nz)), rowsum(cv.abs())
    cnt = rowsum(nz).clamp_min(1.0)
    nb = ld[ci.long()] * nz
    mx = torch.zeros(n, dtype=torch.float64, device=DEV).scatter_reduce_(0, rows, nb, "amax")
    F = torch.stack([ld, sa, rowsum(cv), dg, dg - sa, rowsum(nb) / cnt, mx, rowsum(sa[ci.long()] * nz) / cnt], 1)
    model = warmstart.WarmStartModel.load(device=DEV)
    x = (F - model.mu.double()) * model.inv_sd.double()
    return {"F": F, "y0": _mlp(model.params.double(), model.nin, model.h, x), "pool": F.mean(0).cpu().numpy(),
            "r0": None}
