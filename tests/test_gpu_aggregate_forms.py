"""Algorithm 2 on both sides of each depth at which its path test changes form (ecc(u) = 5 and 9),
for both chunk sizes, unweighted and weighted, against the oracle.  Integer results: equal."""
import numpy as np
import pytest
import torch

import oracle
from paper_2006_13679_amd import api
from paper_2006_13679_amd import graphgen as gg

pytestmark = pytest.mark.gpu


def _graph(ecc):
    """A graph whose vertex 0 has this eccentricity."""
    return gg.complete(7) if ecc == 1 else gg.grid2d(3, ecc - 1) if ecc > 2 else gg.complete_bipartite(3, 5)


@pytest.mark.parametrize("chunk", [4, 8])
@pytest.mark.parametrize("ecc", [1, 2, 3, 4, 5, 6, 8, 9, 10, 11])
def test_counts(ecc, chunk):
    g, T = _graph(ecc), 37
    G = api.Graph.from_host(g.row_ptr, g.col)
    p = api.problem(G, pivot=0, seed=ecc, tau_override=T)
    assert api.bfs(G, p)[2] == ecc
    want = oracle.trees(g.row_ptr, g.col, 0, ecc, 0, T)[2]
    counts, _ = api.flow_counts(G, p, 0, T)
    assert (counts.cpu().numpy() == want).all()
    plan = api.BatchPlan([G], [p], ws=api.Workspace(), schedule=api.Schedule(agg_chunk=chunk))
    plan.execute()
    torch.cuda.synchronize()
    assert (plan.counts[0].cpu().numpy() == want).all()
    plan.close()


@pytest.mark.parametrize("ecc", [4, 5, 6, 9, 10])
def test_weighted_counts(ecc):
    g, T = _graph(ecc), 21
    w = gg.edge_weights(g, ecc, "uniform", 1.0, 4.0)
    G = api.Graph.from_host(g.row_ptr, g.col, weight=w)
    p = api.problem(G, pivot=0, seed=3, tau_override=T)
    _, _, rep = api.diag_lpinv_p(G, p)
    want = oracle.trees_weighted(g.row_ptr, g.col, w, 0, 3, 0, T, rep["fixed_shift"])[2]
    counts, _ = api.flow_counts(G, p, 0, T)
    assert (counts.cpu().numpy() == np.asarray(want)).all()
