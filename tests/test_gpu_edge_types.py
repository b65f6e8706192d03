"""The edge family's kernels in every storage type, with a cost that has off-diagonal entries, on rows short and long
enough for each way a row's neighbours are split over a wave."""

import numpy as np
import pytest
import scipy.sparse as sp
import torch

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def _almbm():
    import paper_2505_15775_amd as m

    return m


# Products of two stored entries and sums over a row or a row's neighbours (at most 300) in the arithmetic type: FP64
# 1e-13 of the sum of magnitudes, float 300 x 2^-24 = 2e-5; a stored gradient is off by half a unit of its last place
# (float 2^-24, bfloat16 2^-9) of the entry.
TOL = {"f64": (1e-13, 2.0 ** -53), "f32": (2e-5, 2.0 ** -24), "bf16": (2e-5, 2.0 ** -9)}


@pytest.mark.parametrize("shape,n,E", [("short", 700, 1503), ("long", 120, 5001), ("dense", 300, 40001)])
@pytest.mark.parametrize("prec", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("r", [1, 3, 4, 5, 8, 11, 16, 24, 32, 48, 64, 100])
def test_edge_kernels(shape, n, E, prec, r):
    rng = np.random.default_rng(r + n)
    iu, ju = np.triu_indices(n, 1)
    pick = np.sort(rng.choice(iu.size, size=E, replace=False))
    ei, ej = iu[pick], ju[pick]
    cp = rng.choice(iu.size, size=2 * n, replace=False)
    w = rng.standard_normal(2 * n)
    S = sp.coo_matrix((np.tile(w, 2), (np.concatenate([iu[cp], ju[cp]]), np.concatenate([ju[cp], iu[cp]]))),
                      shape=(n, n)).tocsr()
    S.sort_indices()
    if prec != "f64":
        S.data = S.data.astype(np.float32).astype(np.float64)
    b, dg = rng.standard_normal(E + 1), rng.standard_normal(n).astype(np.float32).astype(np.float64)
    trace, jc = (0.0, 0.0) if r % 2 else (1.5, 0.5)
    p = _almbm().Problem.edges(n, ei, ej, b, trace, j_coef=jc, cost_csr=(S.indptr, S.indices, S.data), cost_diag=dg,
                               precision=prec, r_max=128, lanczos_kmax=0, device=DEV)
    Rd, Gd = p.factor(rng.standard_normal((n, r))), p.factor(rng.standard_normal((n, r)))
    R, G = Rd.double().cpu().numpy(), Gd.double().cpu().numpy()
    y, s = rng.standard_normal(E + 1), 1.3
    tol, ulp = TOL[prec]

    def amap(A, B):
        edge = 0.5 * ((A[ei] * B[ej]).sum(1) + (B[ei] * A[ej]).sum(1))
        return np.concatenate([[trace * (A * B).sum()], edge])

    def cost(X, absolute=False):
        M, d = (abs(S), np.abs(dg)) if absolute else (S, dg)
        return M @ X + d[:, None] * X + (jc if absolute else -jc) * X.sum(0)[None, :]

    def adjoint(w, X):
        out = trace * w[0] * X
        np.add.at(out, ei, 0.5 * w[1:, None] * X[ej])
        np.add.at(out, ej, 0.5 * w[1:, None] * X[ei])
        return out

    yd = torch.from_numpy(y).to(DEV)
    a = amap(R, R)
    e = a - b
    aa = amap(np.abs(R), np.abs(R))  # magnitudes that rounding is relative to
    for variant in (0, 1):
        p.set_tiles(variant, 0)
        f, Gg, Av = p.objective_grad(Rd, yd, s)
        assert (np.abs(Av.cpu().numpy() - a) <= tol * aa + 1e-300).all()
        # the weights y - s e carry Av's error, the gradient that and its own sums'
        mag = cost(np.abs(R), True) + adjoint(np.abs(y - s * e) + 2 * s * aa, np.abs(R))
        G_o = 2 * (cost(R) - adjoint(y - s * e, R))
        assert (np.abs(Gg.double().cpu().numpy() - G_o) <= 4 * tol * mag + 2 * ulp * np.abs(G_o)).all()
        f_o = (R * cost(R)).sum() + y @ (b - a) + 0.5 * s * (e @ e)
        f_mag = (np.abs(R) * cost(np.abs(R), True)).sum() + np.abs(y) @ aa + s * (np.abs(e) + aa) @ aa
        assert abs(f.item() - f_o) <= 4 * tol * f_mag
        a1, a2 = 2 * amap(R, G), amap(G, G)
        m1, m2 = 2 * amap(np.abs(R), np.abs(G)), amap(np.abs(G), np.abs(G))
        ea = np.abs(e) + aa
        k_o = np.array([f_o, -2 * (G * cost(R)).sum() + y @ a1 - s * (e @ a1),
                        (G * cost(G)).sum() - y @ a2 + 0.5 * s * (a1 @ a1 + 2 * (e @ a2)), -s * (a1 @ a2),
                        0.5 * s * (a2 @ a2)])
        k_mag = np.array([f_mag, 2 * (np.abs(G) * cost(np.abs(R), True)).sum() + np.abs(y) @ m1 + s * (ea @ m1),
                          (np.abs(G) * cost(np.abs(G), True)).sum() + np.abs(y) @ m2 + s * (m1 @ m1 + ea @ m2),
                          s * (m1 @ m2), s * (m2 @ m2)])
        k, _ = p.line_search(Rd, Gd, yd, s)
        assert (np.abs(k.cpu().numpy() - k_o) <= 4 * tol * k_mag).all()
