"""The allocation-free call on graphs whose rows per slot take a large part of the static scratch: the
trees it holds at once, and the sampler without those rows in every form it then takes, against the
CPU oracle.  Integer results: equal, no tolerance.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2006_13679_amd import api
from paper_2006_13679_amd import graphgen as gg

pytestmark = pytest.mark.gpu


def _circulant(n, half, pendants=0):
    """Vertices 0 .. n-1, i joined to i +- d for `half` distances d (1 among them), and `pendants` more
    of degree 1, the j-th on vertex j."""
    d = np.concatenate([[1], np.random.default_rng(4).choice(np.arange(2, n // 2), half - 1, replace=False)])
    cols = (np.arange(n)[:, None] + np.concatenate([d, -d])[None, :]) % n
    cols.sort(axis=1)
    k = pendants
    head = np.concatenate([cols[:k], n + np.arange(k)[:, None]], axis=1)
    col = np.concatenate([head.reshape(-1), cols[k:].reshape(-1), np.arange(k)]).astype(np.int32)
    deg = np.concatenate([np.full(k, 2 * half + 1), np.full(n - k, 2 * half), np.ones(k, dtype=np.int64)])
    return np.concatenate([[0], np.cumsum(deg)]).astype(np.int64), col


def _without_rows(p):
    """Bytes of the workspace less the rows per slot."""
    return api.workspace_bytes(p) - (8 * p.nnz + 255) // 256 * 256


def _call(G, p):
    diag = torch.empty(G.n, dtype=torch.float64, device="cuda")
    counts = torch.empty(G.n, dtype=torch.int64, device="cuda")
    rep = api.diag_lpinv_noalloc_p(G, p, diag, counts)
    return counts.cpu().numpy(), rep


@pytest.mark.parametrize("n,half", [(20_000, 100), (20_000, 155), (40_000, 69), (65_536, 38)])
def test_trees_at_once(n, half):
    """The rows per slot cost the call no more than one tree in ten."""
    row_ptr, col = _circulant(n, half)
    G = api.Graph.from_host(row_ptr, col)
    most = 0
    while most < 300 and _without_rows(api.problem(G, tau_override=300, trees_per_batch=most + 1)) <= api.NOALLOC_SCRATCH_BYTES:
        most += 1
    _, rep = _call(G, api.problem(G, pivot=1, seed=2, tau_override=300, solve_tol=1e-2))
    print(n, len(col), "trees at once", rep["trees_per_batch"], "without the rows", most, flush=True)
    assert 10 * rep["trees_per_batch"] >= 9 * most > 0


# both column widths (the block-split graph has up to 2 n vertices: past the bitmap at 66,000)
@pytest.mark.parametrize("kind,n,half", [("plain", 66_000, 56), ("weighted", 20_000, 100), ("weighted", 66_000, 23),
                                         ("blocks", 20_000, 70), ("blocks", 66_000, 19)])
def test_walks_without_rows_per_slot(kind, n, half):
    row_ptr, col = _circulant(n, half, 40 if kind == "blocks" else 0)
    u, seed, T = 7, 11, 2
    w = gg.edge_weights(gg.Graph(row_ptr, col), 5, "uniform", 1.0, 4.0) if kind == "weighted" else None
    G = api.Graph.from_host(row_ptr, col, weight=w)
    p = api.problem(G, pivot=u, seed=seed, tau_override=T, trees_per_batch=T, solve_tol=1e-2,
                    wilson_variant=api.WILSON_BLOCKS if kind == "blocks" else api.WILSON_PLAIN)
    assert api.workspace_bytes(p) > api.NOALLOC_SCRATCH_BYTES >= _without_rows(p)
    counts, rep = _call(G, p)
    if kind == "weighted":
        _, steps, want = oracle.trees_weighted(row_ptr, col, w, u, seed, 0, T, rep["fixed_shift"], want_parents=False)
    else:
        trees = oracle.trees_blocks if kind == "blocks" else oracle.trees
        _, steps, want = trees(row_ptr, col, u, seed, 0, T, want_parents=False)
    assert rep["walk_steps"] == int(np.sum(steps))
    assert (counts == want).all()
