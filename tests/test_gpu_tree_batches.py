"""Algorithm 2 on caller-supplied trees in launches of more than 16 trees: counts against the oracle
for every split that the workspace gives, and a broken array deep in a launch leaves the counts
alone.  Integer results: equal, no tolerance."""
import pytest
import torch

import oracle
from paper_2006_13679_amd import api
from paper_2006_13679_amd import graphgen as gg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("per_batch", [0, 1, 7, 16, 33])
@pytest.mark.parametrize("name", ["rmat10", "grid21x30", "path300"])
def test_counts(name, per_batch):
    g, u = {"rmat10": (gg.rmat(10, 8, 2), 0), "grid21x30": (gg.grid2d(21, 30), 300), "path300": (gg.path(300), 150)}[name]
    T = 70
    print(name, per_batch, flush=True)
    par, _, want = oracle.trees(g.row_ptr, g.col, u, 4, 0, T)
    G = api.Graph.from_host(g.row_ptr, g.col)
    p = api.problem(G, pivot=u, trees_per_batch=per_batch)
    counts = api.tree_counts(G, p, torch.from_numpy(par), ws=api.Workspace())
    assert (counts.cpu().numpy() == want).all()


def test_broken_tree_in_a_large_launch():
    g, u, T = gg.rmat(10, 8, 2), 0, 70
    par, _, _ = oracle.trees(g.row_ptr, g.col, u, 4, 0, T)
    G = api.Graph.from_host(g.row_ptr, g.col)
    p = api.problem(G, pivot=u)
    bad = par.copy()
    v = next(x for x in range(1, g.n) if bad[53][x] != u)
    bad[53][bad[53][v]] = v  # v and its parent: a cycle that does not reach the pivot
    counts = torch.full((g.n,), 9, dtype=torch.int64, device="cuda")
    with pytest.raises(api.UstdError) as e:
        api.tree_counts(G, p, torch.from_numpy(bad), counts=counts)
    assert e.value.status == api.EINVAL
    assert (counts == 9).all()
