"""Kernel edges: grids, remainders and sizes at which a reduction or a tile of
the HIP kernels changes shape, against the FP64 oracle."""

import numpy as np
import pytest
import torch

import gen
import oracle

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def _almbm():
    import paper_2505_15775_amd as m

    return m


def rel(a, b):
    return float(np.linalg.norm(np.asarray(a, np.float64) - b) / max(np.linalg.norm(b), 1e-300))


@pytest.mark.parametrize("blocks", [8, 64, 72, 544, 1088, 4096])
def test_objective_over_partial_row_counts(blocks):
    """The finalizer adds 15 columns of `blocks` rows: fewer than one trip of its threads, whole trips (68 rows,
    544 x 2) and remainders.  Sums of n r products in FP64: 1e-12 relative covers any order at this size."""
    g = gen.er_graph(40000, 90000, 3, "gauss")
    po = oracle.maxcut_sdp(g)
    p = _almbm().Problem.maxcut(g.n, g.ei, g.ej, g.w, precision="f64", r_max=4, lanczos_kmax=0, device=DEV)
    rng = np.random.default_rng(blocks)
    R, y = rng.standard_normal((g.n, 4)), rng.standard_normal(g.n)
    f_o, G_o, a_o, _ = oracle.objective_grad(po, R, y, 1.3)
    p.set_tiles(0, blocks)
    f, G, Av = p.objective_grad(p.factor(R), torch.from_numpy(y).to(DEV), 1.3)
    assert abs(f.item() - f_o) <= 1e-12 * abs(f_o) + 1e-10
    assert rel(G.cpu(), G_o) <= 1e-12 and rel(Av.cpu(), a_o) <= 1e-12
    k, _ = p.line_search(p.factor(R), p.factor(G_o), torch.from_numpy(y).to(DEV), 1.3)
    k_o = oracle.line_search_coeffs(po, R, G_o, y, 1.3)
    np.testing.assert_allclose(k.cpu().numpy(), k_o, rtol=1e-10, atol=1e-10 * float(np.max(np.abs(k_o))))


@pytest.mark.parametrize("n", [2, 7, 127, 129, 1000, 8191, 8193, 32767, 32769, 70001])
@pytest.mark.parametrize("r", [3, 16])
def test_objective_over_default_grids(n, r):
    """Sizes around the lines of the default grid (16 rows a block up to 512 blocks, 64 rows a block above).  FP64
    sums of n r products: 1e-12 relative covers any order."""
    g = gen.er_graph(n, min(3 * n, n * (n - 1) // 2), n, "gauss")
    po = oracle.maxcut_sdp(g)
    p = _almbm().Problem.maxcut(g.n, g.ei, g.ej, g.w, precision="f64", r_max=16, lanczos_kmax=0, device=DEV)
    rng = np.random.default_rng(n + r)
    R, y = rng.standard_normal((n, r)), rng.standard_normal(n)
    f_o, G_o, a_o, _ = oracle.objective_grad(po, R, y, 1.3)
    for _ in range(2):
        f, G, Av = p.objective_grad(p.factor(R), torch.from_numpy(y).to(DEV), 1.3)
        assert abs(f.item() - f_o) <= 1e-12 * abs(f_o) + 1e-10
        assert rel(G.cpu(), G_o) <= 1e-12 and rel(Av.cpu(), a_o) <= 1e-12


@pytest.mark.parametrize("r", [1, 3, 4, 5, 8, 11, 16, 17, 32, 40, 64, 100, 128])
@pytest.mark.parametrize("shape", ["long", "short", "one_edge"])
def test_edge_family_tiles_against_oracle(shape, r):
    """Every tile of the edge kernels, full and with remainder columns, on long rows (a wave per row), on short
    ones and on a single edge; edge counts that leave partial groups.  FP64 sums of at most n r products."""
    rng = np.random.default_rng(r)
    n, E = {"long": (120, 5001), "short": (700, 1503), "one_edge": (5, 1)}[shape]
    iu, ju = np.triu_indices(n, 1)
    pick = np.sort(rng.choice(iu.size, size=E, replace=False))
    ei, ej = iu[pick], ju[pick]
    b = rng.standard_normal(E + 1)
    dg = rng.standard_normal(n)
    trace, j_coef = (0.0, 0.0) if r % 2 else (1.5, 0.5)
    p = _almbm().Problem.edges(n, ei, ej, b, trace, j_coef=j_coef, cost_diag=dg, precision="f64", r_max=128,
                               lanczos_kmax=0, device=DEV)
    R, G, y = rng.standard_normal((n, r)), rng.standard_normal((n, r)), rng.standard_normal(E + 1)

    def amap(A, B):
        edge = 0.5 * ((A[ei] * B[ej]).sum(1) + (B[ei] * A[ej]).sum(1))
        return np.concatenate([[trace * (A * B).sum()], edge])

    def cost(X):
        return dg[:, None] * X - j_coef * X.sum(0)[None, :]

    s, a = 1.3, amap(R, R)
    e = a - b
    w = y - s * e
    adj = trace * w[0] * R
    np.add.at(adj, ei, 0.5 * w[1:, None] * R[ej])
    np.add.at(adj, ej, 0.5 * w[1:, None] * R[ei])
    f_o = (R * cost(R)).sum() + y @ (b - a) + 0.5 * s * (e @ e)
    f, Gg, Av = p.objective_grad(p.factor(R), torch.from_numpy(y).to(DEV), s)
    assert abs(f.item() - f_o) <= 1e-11 * (1 + abs(f_o) + abs(s * (e @ e)))
    assert rel(Gg.cpu(), 2 * (cost(R) - adj)) <= 1e-12 and rel(Av.cpu(), a) <= 1e-12
    a1, a2 = 2 * amap(R, G), amap(G, G)
    k_o = np.array([f_o, -2 * (G * cost(R)).sum() + y @ a1 - s * (e @ a1),
                    (G * cost(G)).sum() - y @ a2 + 0.5 * s * (a1 @ a1 + 2 * (e @ a2)), -s * (a1 @ a2),
                    0.5 * s * (a2 @ a2)])
    k, _ = p.line_search(p.factor(R), p.factor(G), torch.from_numpy(y).to(DEV), s)
    np.testing.assert_allclose(k.cpu().numpy(), k_o, rtol=1e-10, atol=1e-11 * float(np.max(np.abs(k_o))))


@pytest.mark.parametrize("prec,tol", [("f32", 2e-5), ("bf16", 2e-2)])
@pytest.mark.parametrize("r", [1, 3, 7, 11, 13, 23, 31, 47, 100])
def test_odd_ranks_wide_partial_rows(r, prec, tol):
    """Rows whose width no tile fills are read with the widest accesses that fit: every remainder, both storage
    types.  Tolerances: a sum of at most 100 rounded products in float, one bfloat16 rounding of the result."""
    g = gen.er_graph(501, 3000, 7, "gauss")
    po = oracle.maxcut_sdp(g)
    p = _almbm().Problem.maxcut(g.n, g.ei, g.ej, g.w, precision=prec, r_max=128, lanczos_kmax=0, device=DEV)
    rng = np.random.default_rng(r)
    R = p.factor(rng.standard_normal((g.n, r)))
    y = rng.standard_normal(g.n)
    f_o, G_o, a_o, _ = oracle.objective_grad(po, R.double().cpu().numpy(), y, 0.7)
    f, G, Av = p.objective_grad(R, torch.from_numpy(y).to(DEV), 0.7)
    assert rel(G.double().cpu(), G_o) <= tol and rel(Av.cpu(), a_o) <= 2e-5


@pytest.mark.parametrize("n,kmax", [(40, 39), (300, 120), (2000, 17), (2000, 33), (2000, 70), (16384, 40), (16400, 70),
                                    (66000, 20)])
def test_lanczos_step_shapes(n, kmax):
    """Column counts on both sides of 16, 32 and 64, block counts on both sides of the 64 whose partial sums the
    consumer adds, and rows that leave partial blocks, against the same recurrence in NumPy: after m steps theta is
    the smallest Ritz value of the same Krylov space (FP64, full reorthogonalisation: 1e-9 of the spectrum's size)."""
    g = gen.er_graph(n, 4 * n if n > 100 else 100, 3, "gauss")
    po = oracle.maxcut_sdp(g)
    p = _almbm().Problem.maxcut(g.n, g.ei, g.ej, g.w, precision="f64", r_max=4, lanczos_kmax=kmax, device=DEV)
    y = np.random.default_rng(n).standard_normal(n)
    theta, v, resid, iters = p.lanczos_min_eig(torch.from_numpy(y).to(DEV), max_iter=kmax, tol=1e30, seed=5)
    m = min(kmax, 4 if n <= 4096 else 8)
    assert iters == m
    zmat = lambda x: oracle.cost_apply(po, x[:, None])[:, 0] - y * x  # noqa: E731
    vh = v.cpu().numpy()
    assert abs(np.linalg.norm(vh) - 1) <= 1e-12
    scale = np.abs(y).max() + np.abs(g.w).max() * 8
    assert abs(vh @ zmat(vh) - theta) <= 1e-12 * scale
    assert abs(np.linalg.norm(zmat(vh) - theta * vh) - resid) <= 1e-10 * scale
    theta, v, resid, iters = p.lanczos_min_eig(torch.from_numpy(y).to(DEV), max_iter=kmax, tol=0.0, seed=5)
    vh = v.cpu().numpy()
    assert abs(vh @ zmat(vh) - theta) <= 1e-11 * scale
    assert abs(np.linalg.norm(zmat(vh) - theta * vh) - resid) <= 1e-9 * scale
    if n <= 2000 and kmax >= 33:  # four passes of enough columns find the end of the spectrum
        lam = oracle.min_eig(po, y)
        assert lam - 1e-10 * scale <= theta <= lam + max(resid, 1e-10 * scale)
    th, V, rs, basis = p.lanczos_block(torch.from_numpy(y).to(DEV), 3, max_iter=kmax, seed=2)
    Vh = V.cpu().numpy()
    assert np.abs(Vh.T @ Vh - np.eye(3)).max() <= 1e-10
    for k in range(3):
        assert abs(np.linalg.norm(zmat(Vh[:, k]) - th[k] * Vh[:, k]) - rs[k]) <= 1e-9 * scale


@pytest.mark.parametrize("n,kmax", [(520000, 20), (524289, 70), (530001, 33), (600065, 16)])
def test_lanczos_ordered_sums_over_many_row_chunks(n, kmax):
    """Row chunks on both sides of the 128 from which a projection and the next pass's products read the basis once,
    column counts on both sides of 16, 32 and 64, and chunks that end inside a trip of 256 rows.  The recurrence's
    theta is the Rayleigh quotient of its vector only if every projection is right (1e-11 of the spectrum's size)."""
    g = gen.er_graph(n, n, 3, "gauss")
    po = oracle.maxcut_sdp(g)
    p = _almbm().Problem.maxcut(g.n, g.ei, g.ej, g.w, precision="f64", r_max=4, lanczos_kmax=kmax, device=DEV)
    y = np.random.default_rng(n).standard_normal(n)
    theta, v, resid, iters = p.lanczos_min_eig(torch.from_numpy(y).to(DEV), max_iter=kmax, tol=0.0, seed=5)
    zmat = lambda x: oracle.cost_apply(po, x[:, None])[:, 0] - y * x  # noqa: E731
    vh = v.cpu().numpy()
    scale = np.abs(y).max() + np.abs(g.w).max() * 8
    assert kmax <= iters <= 4 * kmax and abs(np.linalg.norm(vh) - 1) <= 1e-12
    assert abs(vh @ zmat(vh) - theta) <= 1e-11 * scale
    assert abs(np.linalg.norm(zmat(vh) - theta * vh) - resid) <= 1e-9 * scale


@pytest.mark.parametrize("h", [16, 32, 64])
@pytest.mark.parametrize("nin,n,nblocks", [(8, 1, 1), (8, 31, 3), (5, 32, 1), (8, 33, 2), (1, 129, 4), (4, 1000, 7),
                                           (8, 4097, 512), (3, 5000, 64)])
def test_warm_start_network_tiles(h, nin, n, nblocks):
    """Tiles of 32 vertices with every kind of remainder, narrow inputs and blocks without rows, against FP64
    autograd.  FP32 products of at most 64 terms in two layers (and sums over n rows for the gradient): 1e-5."""
    from paper_2505_15775_amd import warmstart

    g = torch.Generator().manual_seed(n + h)
    model = warmstart.WarmStartModel(nin=nin, h=h, device=DEV, seed=n)
    model.params += 0.1 * torch.randn(model.params.shape, generator=g).to(DEV)
    model.mu = torch.randn(8, generator=g).to(DEV)
    model.inv_sd = (0.5 + torch.rand(8, generator=g)).to(DEV)
    X, T = torch.randn((n, nin), generator=g).to(DEV), torch.randn(n, generator=g).to(DEV)
    par = model.params.double().requires_grad_()
    x, o, lay = (X.double() - model.mu[:nin].double()) * model.inv_sd[:nin].double(), 0, []
    for k in (nin * h, h, h * h, h, h, 1):
        lay.append(par[o:o + k])
        o += k
    z = torch.relu(x @ lay[0].view(nin, h) + lay[1])
    out = torch.relu(z @ lay[2].view(h, h) + lay[3]) @ lay[4] + lay[5]
    loss_o = ((out - T.double()) ** 2).mean()
    loss_o.backward()

    class Rows:
        pass

    prob = Rows()
    prob.n = n
    y = model.predict_y0(prob, X)
    assert rel(y.cpu(), out.detach().cpu().numpy()) <= 1e-5
    loss, grad = model.loss_grad(X, T, nblocks=nblocks)
    assert abs(loss.item() - loss_o.item()) <= 1e-5 * loss_o.item()
    assert rel(grad.double().cpu(), par.grad.cpu().numpy()) <= 1e-5


@pytest.mark.parametrize("n", [1, 2, 127, 128, 2049, 70001])
def test_warm_start_pool_counts(n):
    """Column means over row counts around the blocks' shares (FP64 sums of FP32 values)."""
    from paper_2505_15775_amd import warmstart

    F = torch.randn((n, 8), generator=torch.Generator().manual_seed(n)).to(DEV)
    np.testing.assert_allclose(warmstart.pooled(F), F.double().mean(0).cpu().numpy(), rtol=1e-12, atol=1e-13)


@pytest.mark.parametrize("prec,tol", [("f64", 1e-13), ("f32", 1e-5), ("bf16", 1e-2)])
@pytest.mark.parametrize("r", [1, 7, 16, 48])
def test_hub_rows_of_every_trip_count(prec, tol, r):
    """Hub rows on both sides of the wide and narrow trips of the hub kernel (its groups take 4 or 16 entries each),
    with a cost skewed enough to spread the row chunks.  Sums of up to 9000 products per row: FP64 1e-13, float 1e-5
    of the largest row, bfloat16 factors exact on input."""
    rng = np.random.default_rng(r)
    degs = [33, 64, 127, 129, 255, 256, 257, 511, 513, 1023, 1025, 2049, 4097, 9000]
    n = 20000
    ei = np.concatenate([np.full(d, h) for h, d in enumerate(degs)])
    ej = np.concatenate([np.sort(rng.choice(n - 100, size=d, replace=False)) + 100 for d in degs])
    g = gen.Graph(n, ei, ej, rng.standard_normal(ei.size))
    po = oracle.maxcut_sdp(g)
    p = _almbm().Problem.maxcut(g.n, g.ei, g.ej, g.w, precision=prec, r_max=48, lanczos_kmax=30, device=DEV)
    assert p.set_hub_threshold(0) == len(degs)
    X = p.factor(rng.standard_normal((n, r)))
    P_o = oracle.cost_apply(po, X.double().cpu().numpy())
    P = p.cost_apply(X).double().cpu().numpy()
    assert np.abs(P - P_o).max() <= tol * np.abs(P_o).max()
    if prec == "f64":
        y = rng.standard_normal(n)
        theta, v, resid, iters = p.lanczos_min_eig(torch.from_numpy(y).to(DEV), max_iter=30, tol=0.0, seed=5)
        vh = v.cpu().numpy()
        z = oracle.cost_apply(po, vh[:, None])[:, 0] - y * vh
        scale = np.abs(P_o).max() + 5
        assert abs(vh @ z - theta) <= 1e-12 * scale and abs(np.linalg.norm(z - theta * vh) - resid) <= 1e-10 * scale


@pytest.mark.parametrize("solver", ["gd", "lbfgs"])
@pytest.mark.parametrize("tol,steps", [(0.0, 1), (0.0, 33), (2e-2, 200)])
def test_inner_steps_around_the_side_block_grid(solver, tol, steps):
    """512 blocks leave a step's totals to a block of the next pass, 520 to a kernel: the same sums in other groups,
    so the same step count and stop reason and, over these FP64 paths, objectives to 1e-9 relative."""
    m = _almbm()
    g = gen.er_graph(9000, 40000, 5, "gauss")
    out = []
    for blocks in (512, 520):
        p = m.Problem.maxcut(g.n, g.ei, g.ej, g.w, precision="f64", r_max=8, lanczos_kmax=0, lbfgs_memory_max=3,
                             device=DEV)
        p.set_tiles(0, blocks)
        rng = np.random.default_rng(7)
        R = p.factor(rng.standard_normal((g.n, 8)) / 3)
        y = torch.zeros(g.n, dtype=torch.float64, device=DEV)
        opts = dict(inner_solver=m._lib.INNER_LBFGS, lbfgs_memory=3) if solver == "lbfgs" else {}
        out.append(p.inner_solve(R, y, tol, steps, sigma=1.0, **opts))
        p.close()
    (n0, flag0, f0), (n1, flag1, f1) = out
    assert n0 == n1 and flag0 == flag1
    assert abs(f0 - f1) <= 1e-9 * abs(f1)


@pytest.mark.parametrize("r", [3, 8, 33])
@pytest.mark.parametrize("trace,j_coef", [(0.0, 0.0), (1.5, 0.0), (1.5, 0.5)])
def test_edge_family_steps_against_single_calls(r, trace, j_coef):
    """Inner steps, whose pass 3 finalizes passes 1 and 2, against the same steps made of objective, line search and
    an update outside.  Six FP64 gradient steps: rounding of 1e-16 grows by far less than 1e6."""
    rng = np.random.default_rng(r)
    n, E = 900, 7001
    iu, ju = np.triu_indices(n, 1)
    pick = np.sort(rng.choice(iu.size, size=E, replace=False))
    p = _almbm().Problem.edges(n, iu[pick], ju[pick], rng.standard_normal(E + 1), trace, j_coef=j_coef,
                               cost_diag=rng.standard_normal(n), precision="f64", r_max=40, lanczos_kmax=0, device=DEV)
    R0, y = rng.standard_normal((n, r)) / 3, torch.from_numpy(rng.standard_normal(E + 1)).to(DEV)
    R = p.factor(R0)
    done, flag, f = p.inner_solve(R, y, 0.0, 6, sigma=1.3)
    S = p.factor(R0)
    for _ in range(6):
        _, G, _ = p.objective_grad(S, y, 1.3)
        _, t = p.line_search(S, G, y, 1.3)
        S = S - t * G
    f_s, _, _ = p.objective_grad(S, y, 1.3)
    assert (done, flag) == (6, 2)
    assert rel(R.cpu(), S.cpu().numpy()) <= 1e-10
    assert abs(f - f_s.item()) <= 1e-10 * abs(f)
