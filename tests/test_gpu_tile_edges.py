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
