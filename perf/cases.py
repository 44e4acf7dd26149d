"""Performance cases: what users of the library have it do, over its real range.

A case names a graph family and size, the call made on it and the options of
the graph handle. Sizes and option values are those of the repository's own
benchmark and tests (R-MAT with the Graph500 parameters and edge factor 16,
uniform random graphs of mean degree 16, 4-neighbour grids with a tenth of the
edges deleted), with ragged sizes between them.

The graphs are drawn on the GPU with torch from the seed alone and handed to
the library as a host CSR, the form its build takes. `prepare` returns the
built graph handle and the sources, which is what a program holds before it
starts asking for distances; `run` is one call.
"""
from __future__ import annotations

import json
import math
import os

import numpy as np
import torch

import paper_2606_05081_amd
from paper_2606_05081_amd import blest

DEVICE = "cuda"
RMAT_A, RMAT_B, RMAT_C = 0.57, 0.19, 0.19
EDGE_FACTOR = 16
GRID_DELETED = 0.10
MAX_EXACT_LEVELS = 1 << 27  # (source, vertex) pairs for which exact() lays out int64 levels
POLICIES = {"heuristic": blest.Policy.HEURISTIC, "plain": blest.Policy.BVSS, "learned": blest.Policy.LEARNED}


def listed():
    return [
        # The smallest call: one traversal of a graph that fits one compute
        # unit's cache. Launch, entry, exit and host return are all of it.
        {"name": "bfs_rmat_4k", "call": "bfs", "family": "rmat", "n": 4096, "policy": "heuristic"},
        # The plain method (bit-slice top-down at every level, no switch) on
        # the small social-graph shape.
        {"name": "bfs_plain_rmat_64k", "call": "bfs", "family": "rmat", "n": 65536, "policy": "plain"},
        # An ordinary single traversal with the default options, ragged size.
        {"name": "bfs_rmat_ragged_1m", "call": "bfs", "family": "rmat", "n": 1000003, "policy": "heuristic"},
        # The headline: scale-22 R-MAT with the installed switch network.
        {"name": "bfs_learned_rmat_4m", "call": "bfs", "family": "rmat", "n": 1 << 22, "policy": "learned"},
        # Road-network shape: thousands of small levels.
        {"name": "bfs_grid_4m", "call": "bfs", "family": "grid", "rows": 2048, "cols": 2048, "policy": "heuristic"},
        # Uniform random graph: no hubs, few levels, no reordering gain.
        {"name": "bfs_er_1m", "call": "bfs", "family": "er", "n": 1 << 20, "policy": "heuristic"},
        # A web or citation graph: arcs one way, bottom-up over the transpose.
        {"name": "bfs_directed_rmat_256k", "call": "bfs", "family": "rmat", "n": 1 << 18, "policy": "heuristic",
         "directed": True},
        # The smallest multi-source call: one batch of 64 on a small graph.
        {"name": "msbfs_64_rmat_16k", "call": "msbfs", "family": "rmat", "n": 16384, "policy": "heuristic",
         "sources": 64, "width": 64},
        # Batched multi-source levels: 960 sources on scale-20 R-MAT in uneven
        # batches of 64, 128, 256 and 512, int16 levels per (source, vertex).
        {"name": "msbfs_uneven_rmat_1m", "call": "msbfs_batched", "family": "rmat", "n": 1 << 20,
         "policy": "heuristic", "sources": 960, "width": 0},
        # Exact closeness of thousands of vertices of scale-18 R-MAT.
        {"name": "closeness_rmat_256k", "call": "closeness", "family": "rmat", "n": 1 << 18, "policy": "heuristic",
         "sources": 8192, "width": 512},
        # Closeness on a graph without hubs with the multi-source switch
        # network, ragged size and ragged last batch.
        {"name": "closeness_learned_er_300k", "call": "closeness", "family": "er", "n": 300007, "policy": "learned",
         "sources": 700, "width": 256},
        # Per-target distance sums on a road-like grid: many levels, few new
        # pairs in each.
        {"name": "far_grid_64k", "call": "far", "family": "grid", "rows": 256, "cols": 250, "policy": "heuristic",
         "sources": 128, "width": 128},
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: any call on any family, sizes spread over their logarithm."""
    call = rng.choice(["bfs", "bfs", "bfs", "msbfs", "closeness", "far"])
    family = rng.choice(["rmat", "rmat", "er", "grid"])
    case = {"call": call, "family": family, "policy": rng.choice(["heuristic", "heuristic", "plain", "learned"])}
    top = 1 << 20 if call == "bfs" else 1 << 18
    if family == "grid":
        top = top if call == "bfs" else 1 << 15
        area = _log_uniform(rng, 1 << 10, top)
        rows = max(2, int(math.sqrt(area) * rng.uniform(0.6, 1.6)))
        case["rows"], case["cols"] = rows, max(2, area // rows)
    else:
        case["n"] = _log_uniform(rng, 1 << 11, top)
        if family == "rmat" and call == "bfs" and rng.random() < 0.25:
            case["directed"] = True
    if call != "bfs":
        case["sources"] = _log_uniform(rng, 16, 1024)
        case["width"] = rng.choice([64, 128, 256, 512])
    return case


# ---- inputs ----------------------------------------------------------------


def _vertices(case):
    return case["rows"] * case["cols"] if case["family"] == "grid" else case["n"]


def _rmat_pairs(n, gen):
    """EDGE_FACTOR * n R-MAT samples; ids of the next power of two fold back onto n vertices."""
    scale = max(1, math.ceil(math.log2(n)))
    count = EDGE_FACTOR * n
    u = torch.zeros(count, dtype=torch.int64, device=DEVICE)
    v = torch.zeros(count, dtype=torch.int64, device=DEVICE)
    for _ in range(scale):
        r = torch.rand(count, generator=gen, device=DEVICE)
        down = r >= RMAT_A + RMAT_B
        right = ((r >= RMAT_A) & ~down) | (r >= RMAT_A + RMAT_B + RMAT_C)
        u = 2 * u + down
        v = 2 * v + right
    relabel = torch.randperm(1 << scale, generator=gen, device=DEVICE)
    return relabel[u] % n, relabel[v] % n


def _grid_pairs(rows, cols, gen):
    ids = torch.randperm(rows * cols, generator=gen, device=DEVICE).view(rows, cols)
    u = torch.cat([ids[:, :-1].reshape(-1), ids[:-1, :].reshape(-1)])
    v = torch.cat([ids[:, 1:].reshape(-1), ids[1:, :].reshape(-1)])
    keep = torch.rand(u.numel(), generator=gen, device=DEVICE) >= GRID_DELETED
    return u[keep], v[keep]


def _er_pairs(n, gen):
    count = EDGE_FACTOR * n // 2
    return (torch.randint(n, (count,), generator=gen, device=DEVICE),
            torch.randint(n, (count,), generator=gen, device=DEVICE))


def _graph(case, seed):
    """The case's graph as (row_ptr, col, sources): int64 tensors on the GPU, sorted simple rows."""
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(seed)
    n = _vertices(case)
    if case["family"] == "rmat":
        u, v = _rmat_pairs(n, gen)
    elif case["family"] == "grid":
        u, v = _grid_pairs(case["rows"], case["cols"], gen)
    else:
        u, v = _er_pairs(n, gen)
    if not case.get("directed"):
        u, v = torch.cat([u, v]), torch.cat([v, u])
    key = torch.unique((u * n + v)[u != v])
    col = key % n
    degree = torch.bincount(key // n, minlength=n)
    row_ptr = torch.zeros(n + 1, dtype=torch.int64, device=DEVICE)
    row_ptr[1:] = torch.cumsum(degree, 0)
    eligible = torch.nonzero(degree > 0).view(-1)
    pick = torch.randint(eligible.numel(), (case.get("sources", 1),), generator=gen, device=DEVICE)
    return row_ptr, col, eligible[pick]


def _install(g, name, setter):
    path = os.path.join(os.path.dirname(paper_2606_05081_amd.__file__), name)
    with open(path) as f:
        m = json.load(f)
    setter(np.array(m["params"], np.float32), np.array(m["mean"], np.float32), np.array(m["std"], np.float32),
           m.get("min_confidence", 0.5))


def prepare(case, seed):
    row_ptr, col, srcs = _graph(case, seed)
    opts = {"policy": POLICIES[case["policy"]], "directed": int(bool(case.get("directed")))}
    if case.get("width"):
        opts["msbfs_width"] = case["width"]
    g = blest.Graph(row_ptr.to(torch.int32).cpu().numpy(), col.to(torch.int32).cpu().numpy(), **opts)
    if case["policy"] == "learned":
        _install(g, "switch_model.json", g.set_switch_model)
        _install(g, "switch_model_ms.json", g.set_ms_switch_model)
    return {"call": case["call"], "graph": g, "sources": srcs.to(torch.int32).cpu().numpy()}


def run(state):
    g, srcs = state["graph"], state["sources"]
    if state["call"] == "bfs":
        return g.bfs(int(srcs[0]))
    if state["call"] == "msbfs":
        return g.msbfs(srcs)
    if state["call"] == "msbfs_batched":
        return g.msbfs_batched(srcs, [64, 128, 256, 512])
    if state["call"] == "closeness":
        return g.closeness(srcs)
    return g.far(srcs)


# ---- what a pass cannot do without, and its value in 64 bits ----------------


def _arcs(case):
    """Expected arcs of the case's graph (duplicates and self loops removed)."""
    n = _vertices(case)
    if case["family"] == "grid":
        return 2 * (1 - GRID_DELETED) * (2 * n - case["rows"] - case["cols"])
    if case["family"] == "er":
        return EDGE_FACTOR * n * (1 - EDGE_FACTOR / (2 * n))
    duplicates = 0.258 * 0.84 ** (math.log2(n) - 12)
    return (1 if case.get("directed") else 2) * EDGE_FACTOR * n * max(0.4, 1 - duplicates)


def work(case):
    """The graph read once (row pointers and column ids, 4 bytes each), the outputs written once."""
    n = _vertices(case)
    k = case.get("sources", 1)
    out = {"bfs": 4 * n, "msbfs": 2 * k * n, "msbfs_batched": 2 * k * n, "closeness": 24 * k, "far": 8 * n}
    return {"bytes": int(4 * (n + 1) + 4 * _arcs(case) + out[case["call"]]), "flops": 0}


def _levels(row_ptr, col, srcs, n):
    """Hop distances [len(srcs), n], -1 unreached: one sweep over all arcs per level."""
    k = srcs.numel()
    # in-arcs: sort the arcs by head
    tail = torch.repeat_interleave(torch.arange(n, device=DEVICE), row_ptr[1:] - row_ptr[:-1])
    head, order = torch.sort(col)
    tail = tail[order]
    ends = torch.cumsum(torch.bincount(head, minlength=n), 0)
    level = torch.full((k, n), -1, dtype=torch.int64, device=DEVICE)
    rows = torch.arange(k, device=DEVICE)
    level[rows, srcs] = 0
    frontier = torch.zeros((k, n), dtype=torch.int64, device=DEVICE)
    frontier[rows, srcs] = 1
    step = 0
    while True:
        step += 1
        total = torch.zeros((k, tail.numel() + 1), dtype=torch.int64, device=DEVICE)
        torch.cumsum(frontier[:, tail], 1, out=total[:, 1:])
        upto = total[:, ends]
        upto[:, 1:] -= upto[:, :-1].clone()
        new = (upto > 0) & (level < 0)
        if not bool(new.any()):
            return level
        level[new] = step
        frontier = new.to(torch.int64)


def exact(case, seed):
    n = _vertices(case)
    k = case.get("sources", 1)
    if case["call"].startswith("msbfs") and k * n > MAX_EXACT_LEVELS:
        return None
    row_ptr, col, srcs = _graph(case, seed)
    chunk = max(1, min(k, (1 << 28) // max(1, col.numel())))
    parts, sums, reach = [], [], []
    far = torch.zeros(n, dtype=torch.int64, device=DEVICE)
    for s in srcs.split(chunk):
        level = _levels(row_ptr, col, s, n)
        if case["call"] in ("bfs", "msbfs", "msbfs_batched"):
            parts.append(level)
        elif case["call"] == "closeness":
            sums.append(level.clamp(min=0).sum(1))
            reach.append((level >= 0).sum(1))
        else:
            far += level.clamp(min=0).sum(0)
    if case["call"] == "bfs":
        return parts[0][0]
    if case["call"].startswith("msbfs"):
        return torch.cat(parts)
    if case["call"] == "closeness":
        s, r = torch.cat(sums), torch.cat(reach)
        cc = torch.where(s > 0, (r - 1).double() / s.clamp(min=1).double(), torch.zeros_like(s, dtype=torch.float64))
        return s, r, cc
    return far
