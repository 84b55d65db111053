"""Walks that run past their record, one at a time, in every form their chain of rows takes, against
the CPU oracle: rows packed in LDS, columns and row pointers in LDS (the packed rows do not fit),
rows per slot in the workspace (tree state in LDS and in the records, unit weights and
conductances, the block-split graph), and columns and row pointers where a static scratch does not
hold the rows.  Integer results: equal, no tolerance.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2006_13679_amd import api
from paper_2006_13679_amd import graphgen as gg

pytestmark = pytest.mark.gpu


def _circulant(n, half, seed):
    """Vertex i joined to i +- d for `half` distances d: degree 2 half, connected (d = 1)."""
    rng = np.random.default_rng(seed)
    d = np.concatenate([[1], rng.choice(np.arange(2, n // 2), half - 1, replace=False)])
    cols = (np.arange(n)[:, None] + np.concatenate([d, -d])[None, :]) % n
    cols.sort(axis=1)
    return np.arange(n + 1, dtype=np.int64) * (2 * half), cols.astype(np.int32).reshape(-1)


# n: 400 packed rows in LDS; 1600 columns and row pointers in LDS; 4096, 66049 (int32 columns) rows
# in the workspace; 132860 tree state in the records
@pytest.mark.parametrize("rows,cols,T", [(20, 20, 9), (40, 40, 7), (64, 64, 5), (257, 257, 2), (365, 364, 1)])
def test_grids(rows, cols, T):
    g = gg.grid2d(rows, cols)
    u = (rows // 2) * cols + cols // 2
    print("grid", rows, cols, "trees", T, flush=True)
    G = api.Graph.from_host(g.row_ptr, g.col)
    want_par, want_steps, _ = oracle.trees(g.row_ptr, g.col, u, 91, 3, T, want_counts=False)
    p = api.problem(G, pivot=u, seed=91, tau_override=T)
    parents, steps = api.sample_trees(G, p, 3, T)
    assert (steps.cpu().numpy() == want_steps).all()
    assert (parents.cpu().numpy() == want_par).all()


def test_weighted_grid_in_a_batch():
    g = gg.grid2d(36, 31)
    u, T = 500, 6
    w = gg.edge_weights(g, 3, "lognormal")
    G = api.Graph.from_host(g.row_ptr, g.col, weight=w)
    _, want_steps, _ = oracle.trees_weighted(g.row_ptr, g.col, w, u, 5, 0, T, 40, want_acc=False)
    for layout in (api.LAYOUT_AUTO, api.LAYOUT_RECORDS):
        p = api.problem(G, pivot=u, seed=5, tau_override=T)
        plan = api.BatchPlan([G], [p], ws=api.Workspace(), schedule=api.Schedule(layout=layout))
        for _ in range(2):
            plan.execute()
            assert plan.reports()[0]["walk_steps"] == int(np.sum(want_steps))
        plan.close()


def test_static_scratch_without_rows_per_slot():
    n, half = 50_000, 64  # 51 MB of rows per slot beside 13 MB of columns and 6 MB more: past 64 MiB
    row_ptr, col = _circulant(n, half, 4)
    G = api.Graph.from_host(row_ptr, col)
    u, T = 77, 2
    _, want_steps, want_counts = oracle.trees(row_ptr, col, u, 8, 0, T)
    p = api.problem(G, pivot=u, seed=8, tau_override=T)
    diag = torch.empty(n, dtype=torch.float64, device="cuda")
    counts = torch.empty(n, dtype=torch.int64, device="cuda")
    rep = api.diag_lpinv_noalloc_p(G, p, diag, counts)
    assert rep["walk_steps"] == int(want_steps.sum())
    assert (counts.cpu().numpy() == want_counts).all()
