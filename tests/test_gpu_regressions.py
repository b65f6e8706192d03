"""Calls that an earlier change of the kernels or of the host path answered wrongly, refused or slowed down."""

import numpy as np
import pytest
import torch

import gen
import oracle

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
NO_LIMIT = 2 ** 31 - 1


def _almbm():
    import paper_2505_15775_amd as m

    return m


@pytest.mark.parametrize("family,solver", [("diag", "gd"), ("diag", "lbfgs"), ("edges", "gd")])
def test_inner_steps_without_a_limit(family, solver):
    """The largest step limit: a subproblem whose stop test holds at once, and one that takes some steps, end as
    with a limit that is merely large."""
    m = _almbm()
    g = gen.er_graph(500, 2000, 3, "gauss")
    if family == "diag":
        p = m.Problem.maxcut(g.n, g.ei, g.ej, g.w, precision="f64", r_max=8, lanczos_kmax=0, lbfgs_memory_max=3,
                             device=DEV)
    else:
        p = m.Problem.edges(g.n, g.ei, g.ej, np.zeros(g.ei.size + 1), 0.0, cost_diag=np.full(g.n, 0.5),
                            precision="f64", r_max=8, lanczos_kmax=0, device=DEV)
    opts = dict(inner_solver=m._lib.INNER_LBFGS, lbfgs_memory=3) if solver == "lbfgs" else {}
    y = torch.zeros(p.m, dtype=torch.float64, device=DEV)
    R0 = np.random.default_rng(1).standard_normal((g.n, 8)) / 3
    for tol in (1e30, 0.5):
        ends = []
        for limit in (100000, NO_LIMIT):
            R = p.factor(R0)
            ends.append(p.inner_solve(R, y, tol, limit, sigma=1.0, **opts) + (R.cpu().numpy().tobytes(),))
        assert ends[0] == ends[1] and ends[0][1] == 1


def test_batch_steps_without_a_limit():
    m = _almbm()
    gs = [gen.cycle_graph(9), gen.er_graph(400, 1500, 2, "pm1")]
    probs = [m.Problem.maxcut(g.n, g.ei, g.ej, g.w, precision="f64", r_max=16, lanczos_kmax=20, device=DEV) for g in gs]
    batch = m.Batch(probs, rank_stride=16)
    factors = [gen.init_factor(g.n, 4, 1) for g in gs]
    ends = []
    for limit in (100000, NO_LIMIT):
        st, sts, res, R, ranks, y = batch.solve(factors, eps_kkt=1e-2, max_outer=2, max_inner=limit)
        ends.append((st, sts, ranks, [r["inner_total"] for r in res], R.cpu().numpy().tobytes()))
    assert ends[0] == ends[1]


def _bits(p, R, y):
    """Five totals of the rows (those of the line search), whose last bits follow the grid."""
    f, G, _ = p.objective_grad(R, y, 1.3)
    return p.line_search(R, G, y, 1.3)[0].cpu().numpy().tobytes()


@pytest.mark.parametrize("kind", ["skewed", "skewed_f32", "dense_edges", "plain"])
def test_default_grid_of_a_handle(kind):
    """row_blocks = 0 gives the grid that the handle was made with (sums in the same order, so the same bits), also
    where that depends on the row lengths; so does a change of the hub rows and back."""
    m = _almbm()
    rng = np.random.default_rng(3)
    if kind == "dense_edges":
        n = 2000
        iu, ju = np.triu_indices(n, 1)
        pick = np.sort(rng.choice(iu.size, size=40000, replace=False))
        p = m.Problem.edges(n, iu[pick], ju[pick], np.zeros(40001), 0.0, cost_diag=np.full(n, 0.5), precision="f64",
                            r_max=16, lanczos_kmax=0, device=DEV)
    else:
        g = gen.er_graph(70000, 200000, 3, "gauss") if kind == "plain" else gen.rmat_graph(17, 8, 5, "gauss")
        p = m.Problem.maxcut(g.n, g.ei, g.ej, g.w, precision="f32" if kind == "skewed_f32" else "f64", r_max=16,
                             lanczos_kmax=0, device=DEV)
    R = p.factor(rng.standard_normal((p.n, 16)))
    y = torch.from_numpy(rng.standard_normal(p.m)).to(DEV)
    fresh = _bits(p, R, y)
    p.set_tiles(0, 64)
    p.set_tiles(0, 0)
    assert _bits(p, R, y) == fresh
    if kind.startswith("skewed"):
        assert p.set_hub_threshold(-1) == 0
        off = _bits(p, R, y)
        p.set_tiles(0, 0)
        assert _bits(p, R, y) == off
        assert p.set_hub_threshold(0) > 0
        assert _bits(p, R, y) == fresh
        p.set_tiles(0, 64)
        few = _bits(p, R, y)
        p.set_hub_threshold(-1)
        p.set_hub_threshold(0)
        assert _bits(p, R, y) == few  # a grid that the caller chose stays


@pytest.mark.parametrize("n,r,prec", [(511, 5, "f64"), (513, 5, "f64"), (8191, 5, "f64"), (70001, 5, "f64"),
                                      (70001, 24, "bf16"), (70001, 40, "f32"), (262145, 5, "f64"), (300001, 8, "bf16"),
                                      (530000, 3, "f32")])
def test_product_on_either_grid(n, r, prec):
    """C X with and without <X, C X>: the same rows on both grids (sizes around 64 rows a block, 1024 blocks and
    4096, and those where only one grid is used), against the oracle.  Sums of a few products of exact entries: FP64
    1e-13 of the largest, float 1e-6."""
    m = _almbm()
    g = gen.er_graph(n, 3 * n, 3, "gauss")
    p = m.Problem.maxcut(g.n, g.ei, g.ej, g.w, precision=prec, r_max=r, lanczos_kmax=0, device=DEV)
    X = p.factor(np.random.default_rng(n).standard_normal((n, r)))
    P_o = oracle.cost_apply(oracle.maxcut_sdp(g), X.double().cpu().numpy())
    P = p.cost_apply(X).cpu().numpy()
    Q, xpx = p.cost_apply(X, want_xpx=True)
    tol = 1e-13 if prec == "f64" else 1e-6
    assert np.abs(P - P_o).max() <= tol * np.abs(P_o).max()
    assert P.tobytes() == Q.cpu().numpy().tobytes()
    terms = X.double().cpu().numpy() * P_o
    assert abs(xpx.item() - terms.sum()) <= 10 * tol * np.abs(terms).sum()


def test_features_beside_the_handles_other_calls():
    """The feature pass shares no workspace with the handle's other calls: on two streams at once, both give what
    they give alone, bit for bit."""
    from paper_2505_15775_amd import warmstart

    m = _almbm()
    g = gen.er_graph(300000, 1500000, 3, "gauss")
    p = m.Problem.maxcut(g.n, g.ei, g.ej, g.w, precision="f64", r_max=8, lanczos_kmax=0, device=DEV)
    R0 = p.factor(np.random.default_rng(1).standard_normal((g.n, 8)) / 3)
    y = torch.zeros(g.n, dtype=torch.float64, device=DEV)
    F0, steps = warmstart.features(p), 20
    R1 = R0.clone()
    for _ in range(steps):
        p.gd_step(R1, y, 1.0)
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    for _ in range(4):
        R = R0.clone()
        torch.cuda.synchronize()
        Fs = []
        for k in range(steps):
            p.gd_step(R, y, 1.0, stream=s2)
            with torch.cuda.stream(s1):
                Fs += [warmstart.features(p), warmstart.features(p)]
        torch.cuda.synchronize()
        assert torch.equal(R, R1)
        assert all(torch.equal(F, F0) for F in Fs)


def test_stream_of_a_call():
    """The raw handle that calls get is the one of the current stream, or of the stream given."""
    m = _almbm()
    side = torch.cuda.Stream()
    assert m._stream() == torch.cuda.current_stream().cuda_stream
    assert m._stream(side) == side.cuda_stream
    with torch.cuda.stream(side):
        assert m._stream() == side.cuda_stream == torch.cuda.current_stream().cuda_stream


@pytest.mark.parametrize("blocks", [368, 504])
def test_edge_totals_in_a_block_or_a_kernel(blocks):
    """A long table of partial sums (104 a block) is added by a kernel, a shorter one by a block of the line-search
    pass: either way the steps are those of the single calls.  Four FP64 steps: 1e-10 as for the other edge steps."""
    rng = np.random.default_rng(blocks)
    n, r = 4000, 100
    g = gen.er_graph(n, 9000, 3)
    p = _almbm().Problem.edges(n, g.ei, g.ej, rng.standard_normal(9001), 1.5, j_coef=0.5,
                               cost_diag=rng.standard_normal(n), precision="f64", r_max=r, lanczos_kmax=0, device=DEV)
    p.set_tiles(0, blocks)
    R0, y = rng.standard_normal((n, r)) / 10, torch.from_numpy(rng.standard_normal(9001)).to(DEV)
    R, S = p.factor(R0), p.factor(R0)
    assert p.inner_solve(R, y, 0.0, 4, sigma=1.3)[:2] == (4, 2)
    for _ in range(4):
        _, G, _ = p.objective_grad(S, y, 1.3)
        S = S - p.line_search(S, G, y, 1.3)[1] * G
    assert (R - S).norm() <= 1e-10 * S.norm()


@pytest.mark.parametrize("blocks", [2048, 2056])
def test_direction_totals_in_a_block_or_a_kernel(blocks):
    """L-BFGS steps on both sides of the grid up to which a block of the product adds the direction's totals, against
    the default grid: other sums, the same path to 1e-9 over eight FP64 steps."""
    m = _almbm()
    g = gen.er_graph(17000, 60000, 5, "gauss")
    ends = []
    for nb in (0, blocks):
        p = m.Problem.maxcut(g.n, g.ei, g.ej, g.w, precision="f64", r_max=8, lanczos_kmax=0, lbfgs_memory_max=3,
                             device=DEV)
        p.set_tiles(0, nb)
        R = p.factor(np.random.default_rng(7).standard_normal((g.n, 8)) / 3)
        y = torch.zeros(g.n, dtype=torch.float64, device=DEV)
        ends.append(p.inner_solve(R, y, 0.0, 8, sigma=1.0, inner_solver=m._lib.INNER_LBFGS, lbfgs_memory=3))
    assert ends[0][:2] == ends[1][:2] == (8, 2)
    assert abs(ends[0][2] - ends[1][2]) <= 1e-9 * abs(ends[0][2])


@pytest.mark.parametrize("n,r", [(65537, 1), (70001, 3), (85003, 6), (100000, 5), (115001, 7), (160001, 5), (200003, 2),
                                 (300001, 7), (530003, 3)])
def test_narrow_rows_on_the_grid_of_a_call(n, r):
    """Ranks whose rows hold one column per lane, over the grids that a single call takes for them (whole trips, 64
    rows a block, the default): evaluation, line search and gradient step against the oracle, and the handle-free
    evaluation with the same bits.  FP64 sums of n r products: 1e-12 relative covers any order."""
    m = _almbm()
    g = gen.er_graph(n, 3 * n, 3, "gauss")
    po = oracle.maxcut_sdp(g)
    p = m.Problem.maxcut(g.n, g.ei, g.ej, g.w, precision="f64", r_max=8, lanczos_kmax=0, device=DEV)
    rng = np.random.default_rng(n)
    R, D, y = rng.standard_normal((n, r)), rng.standard_normal((n, r)), rng.standard_normal(n)
    Rd, yd = p.factor(R), torch.from_numpy(y).to(DEV)
    f_o, G_o, a_o, _ = oracle.objective_grad(po, R, y, 1.3)
    f, G, Av = p.objective_grad(Rd, yd, 1.3)
    assert abs(f.item() - f_o) <= 1e-12 * abs(f_o) + 1e-10
    assert np.linalg.norm(G.cpu().numpy() - G_o) <= 1e-12 * np.linalg.norm(G_o)
    assert np.linalg.norm(Av.cpu().numpy() - a_o) <= 1e-12 * np.linalg.norm(a_o)
    f2, G2, Av2 = torch.zeros_like(f), torch.zeros_like(G), torch.zeros_like(Av)
    m.objective_grad_noalloc(p.desc, Rd, yd, 1.3, f2, G2, Av2)
    assert f2.item() == f.item() and torch.equal(G2, G) and torch.equal(Av2, Av)
    k, _ = p.line_search(Rd, p.factor(D), yd, 1.3)
    k_o = oracle.line_search_coeffs(po, R, D, y, 1.3)
    np.testing.assert_allclose(k.cpu().numpy(), k_o, rtol=1e-10, atol=1e-10 * float(np.max(np.abs(k_o))))
    t = torch.zeros(1, dtype=torch.float64, device=DEV)
    S = Rd.clone()
    p.gd_step(S, yd, 1.3, t=t)
    _, t_ls = p.line_search(Rd, G, yd, 1.3)
    assert abs(t.item() - t_ls.item()) <= 1e-9 * abs(t_ls.item())
    assert (S - (Rd - t_ls * G)).norm() <= 1e-9 * S.norm()
