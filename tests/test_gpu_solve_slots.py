"""The multi-kernel solve engine at the sizes where its grids and row classes change, and its end
rules: against the one-workgroup engine and the oracle's FP64 column.

Tolerance: both stop at a true relative residual of at most 1e-12, and the largest condition number
of the normalised Laplacians here is below 1e3, so the columns agree within 2e-9 of their norm.
"""
import numpy as np
import pytest

import oracle
from paper_2006_13679_amd import api
from paper_2006_13679_amd import graphgen as gg

pytestmark = pytest.mark.gpu

GRAPHS = {
    "P2": lambda: gg.path(2),
    "K5": lambda: gg.complete(5),
    "star5000": lambda: gg.star(5000),  # one heavy row, 5000 of a single entry
    "K1023-bipartite": lambda: gg.complete_bipartite(1, 1023),
    "rmat10": lambda: gg.rmat(10, 16, 1),
    "rmat15": lambda: gg.rmat(15, 16, 1),  # rows of every class, past the one-workgroup size
    "rhg3000": lambda: gg.hyperbolic(3000, 16.0, seed=4),
}


@pytest.mark.parametrize("mode", [api.SOLVE_FP64, api.SOLVE_MIXED])
@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("name", list(GRAPHS))
def test_engines_agree(name, weighted, mode):
    g = GRAPHS[name]()
    print(name, g.n, weighted, mode, flush=True)
    w = gg.edge_weights(g, 1, "uniform", 1.0, 4.0) if weighted else None
    G = api.Graph.from_host(g.row_ptr, g.col, weight=w)
    p = api.problem(G, pivot=0, solve_mode=mode, solve_tol=1e-12)
    xs = []
    for engine in (api.ENGINE_WORKGROUP, api.ENGINE_MULTI):
        x, rep = api.solve_pivot_column(G, api.with_engine(p, engine))
        assert rep["solve_converged"] == 1 and rep["solve_relres"] <= 1e-12
        xs.append(x.cpu().numpy())
    assert np.linalg.norm(xs[0] - xs[1]) <= 2e-9 * np.linalg.norm(xs[0])


@pytest.mark.parametrize("maxit", [1, 2, 7])
def test_iteration_cap(maxit):
    g = gg.rmat(11, 16, 1)
    G = api.Graph.from_host(g.row_ptr, g.col)
    p = api.with_engine(api.problem(G, pivot=0, solve_tol=1e-14, solve_maxit=maxit), api.ENGINE_MULTI)
    _, rep = api.solve_pivot_column(G, p, allow_notconv=True)
    assert rep["solve_iters"] == maxit and rep["solve_converged"] == 0


def test_repeats_are_bit_identical_and_match_the_oracle():
    g = gg.rmat(15, 16, 1)
    G = api.Graph.from_host(g.row_ptr, g.col)
    p = api.with_engine(api.problem(G, pivot=0, solve_tol=1e-12), api.ENGINE_MULTI)
    a = api.solve_pivot_column(G, p)[0]
    for _ in range(3):
        assert (api.solve_pivot_column(G, p)[0] == a).all()
    want = oracle.solve(g.row_ptr, g.col, 0, 1e-12)[0]
    assert np.linalg.norm(a.cpu().numpy() - want) <= 2e-9 * np.linalg.norm(want)
