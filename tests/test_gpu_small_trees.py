"""Algorithm 2 on caller-supplied trees of small graphs: counts against the oracle on both sides of the
size up to which one launch builds the records, deep, flat and mixed trees; arrays that are no trees;
and small values of trees_per_batch, which are not to split a call into batches of their own.  Integer
results: equal, no tolerance.
"""
import time

import numpy as np
import pytest
import torch

import oracle
from paper_2006_13679_amd import api
from paper_2006_13679_amd import graphgen as gg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name,g,u", [
    ("P2", gg.path(2), 1), ("K5", gg.complete(5), 2), ("path1023", gg.path(1023), 0), ("path1024", gg.path(1024), 1023),
    ("path1025", gg.path(1025), 3), ("star1024", gg.star(1024), 5), ("star1025", gg.star(1025), 5),
    ("grid32x32", gg.grid2d(32), 495), ("grid25x41", gg.grid2d(25, 41), 500), ("tree300", gg.random_tree(300, 3), 9)])
def test_counts(name, g, u):
    T = 21
    print(name, flush=True)
    par, _, want = oracle.trees(g.row_ptr, g.col, u, 6, 2, T)
    G = api.Graph.from_host(g.row_ptr, g.col)
    for per_batch in (0, 1, 4):
        p = api.problem(G, pivot=u, trees_per_batch=per_batch)
        counts = api.tree_counts(G, p, torch.from_numpy(par), ws=api.Workspace())
        assert (counts.cpu().numpy() == want).all()


@pytest.mark.parametrize("n", [40, 1024, 1025])
def test_arrays_that_are_no_trees(n):
    g, u = gg.complete_bipartite(3, n - 3), 0
    par, _, _ = oracle.trees(g.row_ptr, g.col, u, 6, 0, 3)
    G = api.Graph.from_host(g.row_ptr, g.col)
    p = api.problem(G, pivot=u)
    for value in (-1, n, n - 1, 1):  # out of range twice, its own parent, and a cycle 1 <-> n - 1
        bad = par.copy()
        bad[1][n - 1] = value
        if value == 1:
            bad[1][1] = n - 1
        counts = torch.full((n,), 9, dtype=torch.int64, device="cuda")
        with pytest.raises(api.UstdError) as e:
            api.tree_counts(G, p, torch.from_numpy(bad), counts=counts)
        assert e.value.status == api.EINVAL
        assert (counts == 9).all()


def test_small_batches_do_not_split_a_call():
    """64 trees of a graph of five vertices: the workspace of two trees a batch holds them all, so the
    call takes about what it takes with a workspace for 64 (32 batches took 13 times that)."""
    g = gg.complete(5)
    G = api.Graph.from_host(g.row_ptr, g.col)
    par = api.sample_trees(G, api.problem(G, tau_override=64), 0, 64)[0]
    counts = torch.zeros(5, dtype=torch.int64, device="cuda")
    ms = {}
    for per_batch in (64, 2):
        p, ws, t = api.problem(G, trees_per_batch=per_batch), api.Workspace(), []
        for _ in range(15):
            t0 = time.perf_counter()
            api.tree_counts(G, p, par, counts=counts, ws=ws)
            t.append(time.perf_counter() - t0)
        ms[per_batch] = float(np.median(t)) * 1e3
    print(ms, flush=True)
    assert ms[2] < 3 * ms[64]
