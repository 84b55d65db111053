"""Sampler commit paths at the sizes where they change, against the CPU oracle: the window of
free starts (256 vertices), the reorder buffer (128 entries), walks past their record (250 steps),
branches past one piece of the retrace (256 vertices), batches whose inner vertices lie among the
starts in flight (grids) and far from them (R-MAT), with the tree state in LDS and in the records.
Integer results: equal, no tolerance.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2006_13679_amd import api
from paper_2006_13679_amd import graphgen as gg

pytestmark = pytest.mark.gpu

GRAPHS = {
    "path700-far": (lambda: gg.path(700), 699, 4),
    "path513-near": (lambda: gg.path(513), 0, 4),
    "cycle255": (lambda: gg.cycle(255), 7, 12),
    "cycle256": (lambda: gg.cycle(256), 128, 12),
    "cycle257": (lambda: gg.cycle(257), 256, 12),
    "grid3x171": (lambda: gg.grid2d(3, 171), 256, 8),
    "grid45": (lambda: gg.grid2d(45), gg.grid_center_pivot(45), 8),
    "star129": (lambda: gg.star(129), 1, 16),
    "K130": (lambda: gg.complete(130), 64, 16),
    "rmat11": (lambda: gg.rmat(11, 12, 3), 0, 12),
    "rhg1200": (lambda: gg.hyperbolic(1200, 10.0, seed=2), 5, 8),
}


@pytest.mark.parametrize("name", list(GRAPHS))
def test_trees_and_counts(name):
    make, u, T = GRAPHS[name]
    g = make()
    print("graph", name, "n", g.n, "trees", T, flush=True)
    G = api.Graph.from_host(g.row_ptr, g.col)
    want_par, want_steps, want_counts = oracle.trees(g.row_ptr, g.col, u, 77, 0, T)
    # tree state in LDS
    p = api.problem(G, pivot=u, seed=77, tau_override=T)
    parents, steps = api.sample_trees(G, p, 0, T)
    assert (steps.cpu().numpy() == want_steps).all()
    assert (parents.cpu().numpy() == want_par).all()
    counts, _ = api.flow_counts(G, p, 0, T)
    assert (counts.cpu().numpy() == want_counts).all()
    # tree state in the records (every member of a batch in that layout)
    plan = api.BatchPlan([G], [p], ws=api.Workspace(), schedule=api.Schedule(layout=api.LAYOUT_RECORDS))
    plan.execute()
    rep = plan.reports()[0]
    torch.cuda.synchronize()
    assert rep["walk_steps"] == int(want_steps.sum())
    assert (plan.counts[0].cpu().numpy() == want_counts).all()
    plan.close()


def test_weighted_walks_past_the_record():
    g = gg.grid2d(40)
    u, T = gg.grid_center_pivot(40), 6
    w = gg.edge_weights(g, 3, "lognormal")
    G = api.Graph.from_host(g.row_ptr, g.col, weight=w)
    want_par, want_steps, _ = oracle.trees_weighted(g.row_ptr, g.col, w, u, 5, 0, T, 40, want_acc=False)
    p = api.problem(G, pivot=u, seed=5)
    parents, steps = api.sample_trees(G, p, 0, T)
    assert (steps.cpu().numpy() == np.asarray(want_steps)).all()
    assert (parents.cpu().numpy() == np.asarray(want_par)).all()
