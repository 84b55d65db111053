"""Performance cases of the UST estimator of diag(L^+): the calls a user's program makes, at the
sizes of the repository's own workloads and over the ranges around them.

A case is a dict of plain values.  `kind` names the entry point:

  diag          api.diag_lpinv_p          the whole estimator (BFS tree, trees, Algorithm 2, solve)
  noalloc       api.diag_lpinv_noalloc_p  the same without a workspace (serving loops)
  batch         api.BatchPlan             a planned batch of mixed graphs, replayed
  edges         api.edge_counts + api.edge_resistances   all-edge effective resistances
  column        api.solve_pivot_column    the pivot column of L^+
  tree_counts   api.tree_counts           Algorithm 2 on the caller's own spanning trees
  sample        api.sample_trees          spanning trees as parent arrays
  centralities  api.centralities          the vertex measures that follow from diag(L^+)

`family` and its sizes name the graph: "rmat" (scale, ef: Graph500 parameters), "grid" (rows,
cols) or "rhg" (random hyperbolic, n points, average degree about 20), built on the GPU with torch.
The sizes fix the graph up to its vertex numbering, so that the outputs of two seeds have one shape;
the seed gives the numbering (within windows that keep a generator's order at large), the weights
and the key of the estimator's random words.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2006_13679_amd import api
from paper_2006_13679_amd import graphgen as gg

RHG_DEGREE = 20.0
PLAIN_TREE_LIMIT = 30_000  # vertices x trees that exact() walks in plain Python (a few seconds)


def listed():
    return [
        # a serving loop's smallest call: a small graph, few trees, no allocation; all latency
        dict(name="small-noalloc", kind="noalloc", family="grid", rows=13, cols=11, tau=64),
        # the smallest benchmark workload: 32 x 32 grid, 1000 trees (deep trees, long walks)
        dict(name="grid32", kind="diag", family="grid", rows=32, cols=32, tau=1000),
        # the mid-size benchmark workload: a small-world graph, tau from the formula at eps 0.3
        dict(name="rmat16", kind="diag", family="rmat", scale=16, ef=16, eps=0.3),
        # the same with conductances in [1, 4)
        dict(name="rmat16-weighted", kind="diag", family="rmat", scale=16, ef=16, eps=0.3, weighted=True),
        # a hyperbolic graph past the sizes whose tree state fits on chip: long walks, deep chains
        dict(name="rhg200k", kind="diag", family="rhg", n=200_003, eps=0.5),
        # the flagship: 2.4 million vertices, 64 million edges (the cap bounds a seed of larger depth)
        dict(name="rmat22", kind="diag", family="rmat", scale=22, ef=16, eps=0.3, tau_cap=8192),
        # many mixed graphs at once, planned and captured once, replayed per pass
        dict(name="batch16", kind="batch", members=16, scale_max=15, side_max=160, tau_cap=1024),
        # effective resistances of all edges from spanning-edge counts, q trees at eps 0.3
        dict(name="edges-rmat16", kind="edges", family="rmat", scale=16, ef=16, eps=0.3),
        # the linear solve alone, to the default target, on the graph that needs many iterations
        dict(name="column-rhg200k", kind="column", family="rhg", n=200_003),
        # Algorithm 2 on 100 trees that the caller brings
        dict(name="tree-counts-rmat15", kind="tree_counts", family="rmat", scale=15, ef=16, trees=100),
        # spanning trees themselves, as parent arrays, past the on-chip tree state
        dict(name="sample-rmat19", kind="sample", family="rmat", scale=19, ef=16, trees=777),
        # farness, closeness, betweenness and the Kirchhoff index of a flagship-sized diagonal
        dict(name="centralities-2.4M", kind="centralities", n=2_394_961),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_graph(rng, scale, side, n):
    family = rng.choice(["rmat", "rmat", "grid", "rhg"])
    if family == "rmat":
        return dict(family="rmat", scale=rng.randint(9, scale), ef=rng.randint(8, 16))
    if family == "grid":
        return dict(family="grid", rows=_log_uniform(rng, 5, side), cols=_log_uniform(rng, 5, side))
    return dict(family="rhg", n=_log_uniform(rng, 1500, n))


def draw(rng):
    kind = rng.choice(["diag", "diag", "diag", "noalloc", "batch", "edges", "column", "tree_counts", "sample",
                       "centralities"])
    if kind == "centralities":
        return dict(kind=kind, n=_log_uniform(rng, 100, 4_000_000))
    if kind == "batch":
        return dict(kind=kind, members=rng.randint(3, 24), scale_max=rng.randint(10, 15),
                    side_max=rng.randint(16, 160), tau_cap=rng.randint(100, 1024))
    if kind == "noalloc":
        g = _draw_graph(rng, 11, 40, 3000)
        return dict(kind=kind, **g, tau=rng.randint(16, 400))
    if kind == "column":
        g = _draw_graph(rng, 19, 300, 300_000)
        return dict(kind=kind, **g, weighted=rng.random() < 0.3, mixed=rng.random() < 0.4)
    if kind == "edges":
        return dict(kind=kind, **_draw_graph(rng, 17, 100, 100_000), eps=round(rng.uniform(0.25, 0.6), 3))
    if kind in ("tree_counts", "sample"):
        g = _draw_graph(rng, 16 if kind == "tree_counts" else 19, 100, 100_000)
        return dict(kind=kind, **g, trees=rng.randint(1, 300), weighted=rng.random() < 0.25)
    g = _draw_graph(rng, 19, 150, 200_000)
    cap = 2048 if g["family"] == "grid" else 8192
    return dict(kind=kind, **g, eps=round(rng.uniform(0.3, 0.9), 3), tau_cap=cap, weighted=rng.random() < 0.25,
                mixed=rng.random() < 0.25)


# ----------------------------------------------------------------------------------------
# graphs, on the GPU
# ----------------------------------------------------------------------------------------
def _canonical(n, a, b):
    """CSR (int64 row pointers, int32 ascending columns) of the component of the largest-degree
    vertex: symmetrised, without self-loops and duplicates, relabelled in increasing ID order."""
    keep = a != b
    a, b = a[keep], b[keep]
    key = torch.unique(torch.cat([a * n + b, b * n + a]))
    a = torch.div(key, n, rounding_mode="floor")
    b = key - a * n
    del key, keep
    ids = torch.arange(n + 1, device=a.device)
    deg = torch.diff(torch.searchsorted(a, ids))
    seen = torch.zeros(n, dtype=torch.bool, device=a.device)
    seen[torch.argmax(deg)] = True
    count = 0
    while int(seen.sum()) != count:
        count = int(seen.sum())
        seen[b[seen[a]]] = True
    new = torch.cumsum(seen, 0) - 1
    inside = seen[a]
    a, b = new[a[inside]], new[b[inside]]
    row_ptr = torch.searchsorted(a, torch.arange(count + 1, device=a.device))
    return row_ptr, b.to(torch.int32)


def _relabel(row_ptr, col, window, gen):
    """The same graph with its IDs shuffled within runs of `window` vertices."""
    n = len(row_ptr) - 1
    new = torch.empty(n, dtype=torch.int64, device="cuda")
    order = torch.arange(n, device="cuda") // window + torch.rand(n, device="cuda", generator=gen, dtype=torch.float64)
    new[torch.argsort(order)] = torch.arange(n, device="cuda")
    rows = torch.repeat_interleave(new, torch.diff(row_ptr))
    key = torch.sort(rows * n + new[col.long()]).values
    rows = torch.div(key, n, rounding_mode="floor")
    row_ptr = torch.searchsorted(rows, torch.arange(n + 1, device="cuda"))
    return row_ptr, (key - rows * n).to(torch.int32)


def _rmat(scale, ef):
    gen = torch.Generator(device="cuda").manual_seed(1)
    m = ef << scale
    src = torch.zeros(m, dtype=torch.int32, device="cuda")
    dst = torch.zeros_like(src)
    for level in range(scale):
        r = torch.rand(m, device="cuda", generator=gen)
        hi = r >= 0.76                                  # quadrants c and d: the source's bit
        lo = ((r >= 0.57) & ~hi) | (r >= 0.95)          # quadrants b and d: the destination's
        src |= hi.to(torch.int32) << level
        dst |= lo.to(torch.int32) << level
    return _canonical(1 << scale, src.long(), dst.long())


def _rhg(n):
    """Random hyperbolic graph, threshold model, power-law exponent 3: points by angle, edges
    found per radial band in the angular window that the band's inner radius admits."""
    gen = torch.Generator(device="cuda").manual_seed(1)
    R = 2.0 * math.log(8.0 * n / (math.pi * RHG_DEGREE))
    theta = torch.sort(torch.rand(n, device="cuda", generator=gen, dtype=torch.float64) * (2.0 * math.pi)).values
    u = torch.rand(n, device="cuda", generator=gen, dtype=torch.float64)
    r = torch.acosh(1.0 + u * (math.cosh(R) - 1.0))
    ch, sh = torch.cosh(r), torch.sinh(r)
    bands = max(4, 2 * math.ceil(math.log2(n)))
    band = torch.clamp((r * (bands / R)).long(), max=bands - 1)
    ea, eb = [], []
    for i in range(bands):
        members = torch.nonzero(band == i).flatten()
        query = torch.nonzero(band >= i).flatten()
        k = len(members)
        if k == 0:
            continue
        cb, sb = math.cosh(R * i / bands), math.sinh(R * i / bands)
        cos_gap = (ch[query] * cb - math.cosh(R)) / torch.clamp(sh[query] * sb, min=1e-300)
        gap = torch.acos(torch.clamp(cos_gap, -1.0, 1.0))
        angle = theta[members]
        ring = torch.cat([angle - 2.0 * math.pi, angle, angle + 2.0 * math.pi])
        first = torch.searchsorted(ring, theta[query] - gap)
        last = torch.searchsorted(ring, theta[query] + gap, right=True)
        cnt = torch.clamp(last - first, max=k)
        q = torch.repeat_interleave(torch.arange(len(query), device="cuda"), cnt)
        at = torch.arange(len(q), device="cuda") - torch.repeat_interleave(torch.cumsum(cnt, 0) - cnt, cnt)
        x, y = query[q], members[(first[q] + at) % k]
        near = ch[x] * ch[y] - sh[x] * sh[y] * torch.cos(theta[x] - theta[y]) < math.cosh(R)
        keep = near & ((band[x] > i) | (x < y))
        ea.append(x[keep])
        eb.append(y[keep])
    return _canonical(n, torch.cat(ea), torch.cat(eb))


def _weights(row_ptr, col, gen):
    """One conductance in [1, 4) per edge, at both of its entries."""
    n = len(row_ptr) - 1
    rows = torch.repeat_interleave(torch.arange(n, device="cuda"), torch.diff(row_ptr))
    key, mirror = rows * n + col, col.long() * n + rows
    w = 1.0 + 3.0 * torch.rand(len(col), device="cuda", generator=gen, dtype=torch.float64)
    return torch.where(rows < col, w, w[torch.searchsorted(key, mirror)])


def _graph(case, seed):
    """The case's graph, and the pivot a user's program gives it (-1: the largest degree)."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    pivot = -1
    if case["family"] == "grid":
        g = gg.grid2d(case["rows"], case["cols"])
        row_ptr = torch.from_numpy(g.row_ptr).cuda()
        col = torch.from_numpy(g.col).cuda()
        pivot = gg.grid_center_pivot(case["rows"], case["cols"])
    elif case["family"] == "rmat":
        # R-MAT IDs carry the degrees (hubs at IDs with few bits set): a shuffle of 32 keeps that
        row_ptr, col = _relabel(*_rmat(case["scale"], case["ef"]), 32, gen)
    else:
        # the points of a hyperbolic graph come in no order
        row_ptr, col = _rhg(case["n"])
        row_ptr, col = _relabel(row_ptr, col, len(row_ptr), gen)
    w = _weights(row_ptr, col, gen) if case.get("weighted") else None
    return api.Graph(row_ptr, col, w), pivot


def _problem(case, seed):
    g, pivot = _graph(case, seed)
    p = api.problem(g, pivot=pivot, eps=case.get("eps", 0.3), seed=seed, tau_override=case.get("tau", 0),
                    tau_cap=case.get("tau_cap", 0),
                    solve_mode=api.SOLVE_MIXED if case.get("mixed") else api.SOLVE_FP64)
    return g, p


def _batch_members(case, seed):
    """Half R-MAT graphs (scale from 10, edge factor 8 to 16), half square grids (side from 16)."""
    rng = np.random.default_rng(case["members"])
    graphs, probs = [], []
    for i in range(case["members"]):
        if i < case["members"] // 2:
            c = dict(family="rmat", scale=int(rng.integers(10, case["scale_max"] + 1)), ef=int(rng.integers(8, 17)))
        else:
            side = int(rng.integers(16, case["side_max"] + 1))
            c = dict(family="grid", rows=side, cols=side)
        g, p = _problem(dict(c, tau_cap=case["tau_cap"]), seed + 1000 * i)
        graphs.append(g)
        probs.append(p)
    return graphs, probs


# ----------------------------------------------------------------------------------------
# the cases
# ----------------------------------------------------------------------------------------
def prepare(case, seed):
    kind = case["kind"]
    if kind == "centralities":
        gen = torch.Generator(device="cuda").manual_seed(seed)
        # diagonals of small-world graphs: about 1/degree, degrees of a power law
        u = torch.rand(case["n"], device="cuda", generator=gen, dtype=torch.float64)
        return dict(kind=kind, diag=0.01 + u * u)
    if kind == "batch":
        graphs, probs = _batch_members(case, seed)
        plan = api.BatchPlan(graphs, probs, ws=api.Workspace())
        plan.capture()
        return dict(kind=kind, plan=plan)
    g, p = _problem(case, seed)
    state = dict(kind=kind, g=g, p=p)
    if kind == "noalloc":
        state["diag"] = torch.empty(g.n, dtype=torch.float64, device="cuda")
        state["counts"] = torch.empty(g.n, dtype=torch.int64, device="cuda")
    elif kind == "edges":
        state["q"] = api.edge_sample_size(g.n, g.nnz // 2, case["eps"])
    elif kind == "sample":
        state["trees"] = case["trees"]
    elif kind == "tree_counts":
        state["parents"] = api.sample_trees(g, p, 0, case["trees"])[0]
    return state


def run(state):
    kind = state["kind"]
    if kind == "centralities":
        return api.centralities(state["diag"])
    if kind == "batch":
        plan = state["plan"]
        plan.replay()
        return dict(diags=plan.diags, counts=plan.counts)
    g, p = state["g"], state["p"]
    if kind == "diag":
        diag, counts, rep = api.diag_lpinv_p(g, p)
        return dict(diag=diag, counts=counts, walk_steps=rep["walk_steps"])
    if kind == "noalloc":
        rep = api.diag_lpinv_noalloc_p(g, p, state["diag"], state["counts"])
        return dict(diag=state["diag"], counts=state["counts"], walk_steps=rep["walk_steps"])
    if kind == "edges":
        counts, rep = api.edge_counts(g, p, 0, state["q"])
        r, denom = api.edge_resistances(g, counts, state["q"])
        return dict(counts=counts, r=r, denom=denom, walk_steps=rep["walk_steps"])
    if kind == "column":
        return api.solve_pivot_column(g, p)[0]
    if kind == "tree_counts":
        return api.tree_counts(g, p, state["parents"])
    parents, steps = api.sample_trees(g, p, 0, state["trees"])
    return dict(parents=parents, steps=steps)


# ----------------------------------------------------------------------------------------
# work and exact values
# ----------------------------------------------------------------------------------------
def _sizes(case):
    """(n, CSR entries, eccentricity), about what the generators give."""
    if case["family"] == "grid":
        r, c = case["rows"], case["cols"]
        return r * c, 2 * (r * (c - 1) + c * (r - 1)), (r + c) // 2
    if case["family"] == "rmat":
        return int(0.64 * (1 << case["scale"])), int(1.87 * case["ef"] * (1 << case["scale"])), 5
    return case["n"], int(RHG_DEGREE * case["n"]), 8


def _trees(case, n, nnz, ecc):
    if case.get("tau"):
        return case["tau"]
    tau = ecc * ecc * math.ceil(math.log(nnz * n) / (2.0 * 0.49 * case.get("eps", 0.3) ** 2))
    return min(tau, case["tau_cap"]) if case.get("tau_cap") else tau


def work(case):
    """Input read once, output written once; per tree and vertex one walk step at least, with a
    quarter of a Philox4x32-10 block (about 25 operations), a step and a signed count (about 15)."""
    kind = case["kind"]
    if kind == "centralities":
        return dict(bytes=32 * case["n"], flops=8 * case["n"])
    if kind == "batch":
        half = case["members"] // 2
        rm = dict(family="rmat", scale=(10 + case["scale_max"]) // 2, ef=12)
        side = (16 + case["side_max"]) // 2
        gr = dict(family="grid", rows=side, cols=side)
        total = dict(bytes=0, flops=0)
        for c, k in ((rm, half), (gr, case["members"] - half)):
            w = work(dict(c, kind="diag", tau_cap=case["tau_cap"]))
            total = {key: total[key] + k * w[key] for key in total}
        return total
    n, nnz, ecc = _sizes(case)
    graph = 8 * (n + 1) + 4 * nnz + (8 * nnz if case.get("weighted") else 0)
    if kind == "column":  # an operator's read and two operations an entry, once a digit or so
        return dict(bytes=graph + 8 * n, flops=40 * (2 * nnz + 10 * n))
    if kind == "tree_counts":
        return dict(bytes=graph + 4 * n * case["trees"] + 8 * n, flops=15 * n * case["trees"])
    if kind == "sample":
        return dict(bytes=graph + 4 * n * case["trees"], flops=40 * n * case["trees"])
    if kind == "edges":
        q = math.ceil(2.0 * math.log(nnz * n) / case["eps"] ** 2)
        return dict(bytes=graph + 24 * nnz, flops=40 * n * q)
    return dict(bytes=graph + 16 * n, flops=40 * n * _trees(case, n, nnz, ecc))


def _laplacian(g):
    n = g.n
    rows = torch.repeat_interleave(torch.arange(n, device=g.col.device), torch.diff(g.row_ptr))
    w = g.weight if g.weight is not None else torch.ones(g.nnz, dtype=torch.float64, device=g.col.device)
    deg = torch.zeros(n, dtype=torch.float64, device=g.col.device).index_add_(0, rows, w)
    A = torch.sparse_csr_tensor(g.row_ptr, g.col.long(), w, size=(n, n))
    return A, deg


def _pivot_column(g, u):
    """Column u of L^+ by conjugate gradients in 64 bits, restarted on the true residual."""
    A, deg = _laplacian(g)
    b = torch.full((g.n,), -1.0 / g.n, dtype=torch.float64, device=deg.device)
    b[u] += 1.0
    x = torch.zeros_like(b)
    for _ in range(3):
        r = b - (deg * x - A @ x)
        r -= r.mean()
        z = r / deg
        p, rz = z.clone(), torch.dot(r, z)
        start, e = torch.linalg.vector_norm(r), torch.zeros_like(b)
        for it in range(20000):
            q = deg * p - A @ p
            alpha = rz / torch.dot(p, q)
            e += alpha * p
            r -= alpha * q
            if it % 50 == 49 and float(torch.linalg.vector_norm(r) / start) < 1e-10:
                break
            z = r / deg
            rz, old = torch.dot(r, z), rz
            p = z + (rz / old) * p
        x += e
    return x - x.mean()


def _philox(c0, s, t, key):
    c = [c0, s, t & 0xFFFFFFFF, t >> 32]
    k0, k1 = key & 0xFFFFFFFF, key >> 32
    for _ in range(10):
        a, b = 0xD2511F53 * c[0], 0xCD9E8D57 * c[2]
        c = [(b >> 32) ^ c[1] ^ k0, b & 0xFFFFFFFF, (a >> 32) ^ c[3] ^ k1, a & 0xFFFFFFFF]
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    return c


def _plain_counts(g, u, seed, tau):
    """Wilson's algorithm and Algorithm 2 as defined, in plain Python: (counts, walk steps)."""
    rp, col, n = g.row_ptr.tolist(), g.col.tolist(), g.n
    parB, order = [-1] * n, [u]
    dist = [0 if v == u else n for v in range(n)]
    for v in order:
        for y in col[rp[v]:rp[v + 1]]:
            if dist[y] == n:
                dist[y] = dist[v] + 1
                order.append(y)
    for v in range(n):
        if v != u:
            parB[v] = min(y for y in col[rp[v]:rp[v + 1]] if dist[y] == dist[v] - 1)
    counts, steps = [0] * n, 0
    for t in range(tau):
        par = [None] * n
        par[u] = -1
        for s in range(n):
            nxt, x, k, words = {}, s, 0, None
            while par[x] is None:
                if k % 4 == 0:
                    words = _philox(k // 4, s, t, seed)
                y = col[rp[x] + ((words[k % 4] * (rp[x + 1] - rp[x])) >> 32)]
                nxt[x], x, k = y, y, k + 1
            steps += k
            x = s
            while par[x] is None:
                par[x], x = nxt[x], nxt[x]
        for v in range(n):
            path, x = set(), v
            while x != u:
                path.add((x, parB[x]))
                x = parB[x]
            x = v
            while x != u:  # the tree path from v to u: an edge of P(v) forward or backward
                counts[v] += ((x, par[x]) in path) - ((par[x], x) in path)
                x = par[x]
    return counts, steps


def exact(case, seed):
    kind = case["kind"]
    if kind == "centralities":
        d = prepare(case, seed)["diag"].cpu().numpy()
        n, tr = len(d), math.fsum(d.tolist())
        far = n * d + tr
        return dict(farness=far, closeness=(n - 1) / far, nrwb=1.0 / n + tr / ((n - 1) * far), trace=tr,
                    kirchhoff=n * tr)
    if kind == "column":
        g, p = _problem(case, seed)
        u = p.pivot if p.pivot >= 0 else int(torch.argmax(torch.diff(g.row_ptr)))
        return _pivot_column(g, u)
    if kind in ("diag", "noalloc") and case.get("tau") and not case.get("weighted"):
        g, p = _problem(case, seed)
        if g.n * case["tau"] > PLAIN_TREE_LIMIT:
            return None
        u = p.pivot if p.pivot >= 0 else int(torch.argmax(torch.diff(g.row_ptr)))
        counts, steps = _plain_counts(g, u, p.seed, case["tau"])
        x = _pivot_column(g, u).cpu().numpy()
        diag = np.array(counts, dtype=np.float64) / case["tau"] - x[u] + 2.0 * x
        diag[u] = x[u]
        return dict(diag=diag, counts=np.array(counts, dtype=np.int64), walk_steps=steps)
    return None
