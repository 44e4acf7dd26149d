"""Eager levels of one workgroup and the workgroup's list of new vertices, at
the sizes where they hand over: 1,024 frontier vertices and 4,096 frontier edges
bound a level of one workgroup, 4,096 entries its list. Levels are integers
with one correct value, so every comparison is array equality."""
import numpy as np
import pytest

import oracle
from paper_2606_05081_amd import inputs
from tests import helpers as H

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def blest():
    import torch
    from paper_2606_05081_amd import blest as b
    assert torch.cuda.is_available()
    b.lib()
    return b


def layered(widths, extra=0):
    """Levels of the given widths from vertex 0: vertex j of a level hangs on
    vertex j mod w of the level before, and on `extra` further ones of it."""
    base = np.concatenate([[0], np.cumsum(widths)])
    us, vs = [], []
    for i in range(1, len(widths)):
        j = np.arange(widths[i])
        for k in range(extra + 1):
            us.append(base[i - 1] + (j + 37 * k) % widths[i - 1])
            vs.append(base[i] + j)
    return inputs.from_pairs(int(base[-1]), np.concatenate(us), np.concatenate(vs))


CASES = {
    # frontier of 1,023 to 1,025 and about one vertex per thread, then small again
    "frontier": [1, 511, 3, 512, 2, 513, 1, 1023, 5, 1024, 1, 1025, 7, 1100, 3],
    # one level's edges at 4,095 to 4,098 (each vertex also counts its parent)
    "edges": [1, 1, 4094, 1, 4095, 1, 4096, 1, 4097, 1, 7],
    # rows of 8 and 9 columns (the two row walks), 64 and 65 rows per wave
    "rows": [1, 7, 49, 64, 512, 65, 520, 64, 511],
    # many hand-overs in both directions
    "zigzag": [1, 1025, 1, 1025, 1, 4200, 1, 2, 4, 8, 16, 32, 64, 128, 256, 512, 1024, 512, 256, 1],
    # one row longer than a workgroup's list
    "hub": [1, 20000, 1, 20000, 3],
}


@pytest.mark.parametrize("opt", [dict(), dict(sigma=16, reorder=0), dict(sigma=32, block_size=256),
                                 dict(tau=256, block_size=1024), dict(tau=64, reorder=3)])
@pytest.mark.parametrize("name", list(CASES))
def test_episode_edges(blest, name, opt):
    for extra in (0, 2):
        rp, col = layered(CASES[name], extra)
        g = blest.Graph(rp, col, update_scheme=blest.Update.EAGER, **opt)
        b = g.export_bvss()
        for src in (0, (rp.size - 1) // 2, rp.size - 2):
            ref = oracle.bfs(rp, col, src)
            for policy in (blest.Policy.BVSS, blest.Policy.HEURISTIC):
                g.set_policy(policy, 10.0)
                assert np.array_equal(g.bfs(src).cpu().numpy(), ref)
            stats = g.level_stats()
            assert [r["frontier"] for r in stats] == oracle.level_counts(ref).tolist()
            if opt.get("reorder") == 0:
                rep = oracle.switch_replay(ref, rp, b["real_ptrs"], opt.get("sigma", 8), eta=10.0)
                assert [r["queue"] for r in stats] == [r["queue"] for r in rep]
        g.close()


def test_episode_directed(blest):
    # arcs from a level to the next only, hubs among them
    rp, col = layered(CASES["zigzag"], 1)
    n = rp.size - 1
    u = np.repeat(np.arange(n), np.diff(rp))
    keep = u < col
    rpd = np.concatenate([[0], np.cumsum(np.bincount(u[keep], minlength=n))]).astype(rp.dtype)
    g = blest.Graph(rpd, col[keep], directed=1, update_scheme=blest.Update.EAGER)
    for src in (0, 1, n // 2):
        ref = oracle.bfs(rpd, col[keep], src)
        assert np.array_equal(g.bfs(src).cpu().numpy(), ref)
    g.close()
