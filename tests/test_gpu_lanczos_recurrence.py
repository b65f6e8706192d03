"""The Lanczos recurrence of a solve and of alm_bm_lanczos_min_eig, entry by entry, against the same recurrence in
NumPy from the same counter-based start."""

import ctypes as C

import numpy as np
import pytest
import scipy.sparse as sp
import torch

import gen
import oracle

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def _almbm():
    import paper_2505_15775_amd as m

    return m


def start_vector(n, seed):
    """SplitMix64 output of (seed, index) as a uniform in [-1, 1)."""
    with np.errstate(over="ignore"):
        z = np.uint64(seed) * np.uint64(0x9E3779B97F4A7C15) + np.arange(1, n + 1, dtype=np.uint64) * np.uint64(
            0xBF58476D1CE4E5B9)
        z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
        z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
        z = z ^ (z >> np.uint64(31))
    return (z >> np.uint64(11)).astype(np.float64) * 2.0 ** -52 - 1.0


def recurrence(zmat, x, m):
    """(alpha, beta, theta, Ritz vector) after m steps with two classical Gram-Schmidt passes each."""
    Q, al, be = [x / np.linalg.norm(x)], [], []
    for j in range(m):
        B = np.stack(Q, axis=1)
        w = zmat(Q[j])
        h1 = B.T @ w
        w = w - B @ h1
        h2 = B.T @ w
        w = w - B @ h2
        al.append(h1[j] + h2[j])
        be.append(np.linalg.norm(w))
        Q.append(w / be[-1])
    lam, U = np.linalg.eigh(np.diag(al) + np.diag(be[:-1], 1) + np.diag(be[:-1], -1))
    v = np.stack(Q[:m], axis=1) @ U[:, 0]
    return np.array(al), np.array(be), lam[0], v / np.linalg.norm(v)


def diag_problem(n, kmax):
    g = gen.er_graph(n, 4 * n, 3, "gauss")
    po = oracle.maxcut_sdp(g)
    p = _almbm().Problem.maxcut(g.n, g.ei, g.ej, g.w, precision="f64", r_max=4, lanczos_kmax=kmax, device=DEV)
    y = np.random.default_rng(n).standard_normal(n)
    return p, y, lambda x: oracle.cost_apply(po, x[:, None])[:, 0] - y * x


def edge_problem(n, kmax, j_coef):
    """Trace row, 3 n edges, a cost with off-diagonal entries and a diagonal, and a -J term of the other terms' size."""
    rng = np.random.default_rng(n)
    g, s = gen.er_graph(n, 3 * n, 5), gen.er_graph(n, 2 * n, 6, "gauss")
    E = g.ei.size
    S = sp.coo_matrix((np.concatenate([s.w, s.w]), (np.concatenate([s.ei, s.ej]), np.concatenate([s.ej, s.ei]))),
                      shape=(n, n)).tocsr()
    S.sort_indices()
    dg, y = rng.standard_normal(n), rng.standard_normal(E + 1)
    p = _almbm().Problem.edges(n, g.ei, g.ej, np.zeros(E + 1), 1.5, j_coef=j_coef,
                               cost_csr=(S.indptr, S.indices, S.data), cost_diag=dg, precision="f64", r_max=4,
                               lanczos_kmax=kmax, device=DEV)
    A = sp.coo_matrix((np.tile(0.5 * y[1:], 2), (np.concatenate([g.ei, g.ej]), np.concatenate([g.ej, g.ei]))),
                      shape=(n, n)).tocsr()
    return p, y, lambda x: S @ x + (dg - 1.5 * y[0]) * x - j_coef * x.sum() - A @ x


def run(p, y, kmax, tol, restarts, ordered):
    m = _almbm()
    f = m._lib.lib.alm_bm_internal_lanczos
    f.restype = C.c_int32
    f.argtypes = [C.c_void_p, C.c_void_p, C.c_int32, C.c_double, C.c_uint64, C.c_int32, C.c_int32, C.c_void_p,
                  C.c_void_p, C.c_void_p, C.c_void_p]
    v = torch.empty(p.n, dtype=torch.float64, device=DEV)
    yd, tri, out = torch.from_numpy(y).to(DEV), np.zeros(2 * kmax), np.zeros(4)
    m.check(f(p._h, yd.data_ptr(), kmax, tol, 5, restarts, ordered, v.data_ptr(), tri.ctypes.data, out.ctypes.data,
              torch.cuda.current_stream().cuda_stream), "internal_lanczos")
    return tri[:kmax], tri[kmax:], out, v.cpu().numpy()


# Both sides of 16, 32 and 64 columns; 8, 12, 64 and 72 blocks of 256 rows (64: the most whose partial sums the consumer
# adds), 256 of them, and 72 of 1024 rows beyond 65536.
SHAPES = [(1000, 17), (3000, 33), (16384, 40), (16400, 70), (65536, 20), (65537, 20)]


@pytest.mark.parametrize("ordered", [0, 1])
@pytest.mark.parametrize("n,kmax", SHAPES)
@pytest.mark.parametrize("family", ["diag", "edges", "edges_j"])
def test_recurrence_entries(family, n, kmax, ordered):
    """Tolerances, of the size of Z: sums of n products in FP64 are exact to 1e-13, which the first six steps of a
    random start magnify by far less than 100; later steps by up to 1e6 once an end of the spectrum is found (a
    wrong total, buffer or sum of the start is of order one).  The Ritz value is of second order in the basis."""
    if family == "diag":
        p, y, zmat = diag_problem(n, kmax)
    else:
        p, y, zmat = edge_problem(n, kmax, 8.0 / n if family == "edges_j" else 0.0)
    al, be, theta, v = recurrence(zmat, start_vector(n, 5), kmax)
    scale = np.abs(al).max() + 2 * be.max()
    a, b, out, vd = run(p, y, kmax, 0.0, 0, ordered)
    assert out[2] == kmax and out[3] == kmax
    assert max(np.abs(a - al)[:6].max(), np.abs(b - be)[:6].max()) <= 1e-11 * scale
    assert max(np.abs(a - al).max(), np.abs(b - be).max()) <= 1e-6 * scale
    assert abs(out[0] - theta) <= 1e-9 * scale
    assert abs(np.linalg.norm(vd) - 1) <= 1e-12
    assert abs(np.linalg.norm(zmat(vd) - out[0] * vd) - out[1]) <= 1e-9 * scale
    a, b, out, vd = run(p, y, kmax, 0.0, 1, ordered)
    steps = int(out[2]) - kmax  # fewer where the start is a converged Ritz vector and the recurrence breaks down
    assert 1 <= steps <= kmax
    _, _, theta, _ = recurrence(zmat, v, steps)
    assert abs(out[0] - theta) <= 1e-7 * scale
    assert abs(np.linalg.norm(zmat(vd) - out[0] * vd) - out[1]) <= 1e-9 * scale


@pytest.mark.parametrize("ordered", [0, 1])
@pytest.mark.parametrize("n", [1000, 4096, 4097, 20000, 65536, 65537])
def test_steps_past_the_check_that_ends_a_pass(n, ordered):
    """A check is looked at after one more step at most, so that a pass of few steps costs few; the result is that
    of the check's own step count."""
    p, y, zmat = diag_problem(n, 60)
    first = 4 if n <= 4096 else 8
    a, b, out, v = run(p, y, 60, 1e30, 0, ordered)
    assert out[2] == first and out[3] <= first + 1
    al, be, theta, _ = recurrence(zmat, start_vector(n, 5), first)
    assert abs(out[0] - theta) <= 1e-11 * (np.abs(al).max() + 2 * be.max())
    assert abs(v @ zmat(v) - out[0]) <= 1e-11 * (np.abs(al).max() + 2 * be.max())
