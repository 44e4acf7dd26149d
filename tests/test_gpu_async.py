"""opts.async = 1: calls return before the GPU is done and blest_sync reports
the errors of all calls since the last one. A good call, calls back to back (also
multi-source ones, which take their sources with the launch), a failed call
followed by good ones before the sync, and good calls after it."""
import numpy as np
import pytest

import oracle
from paper_2606_05081_amd import inputs
from tests import helpers as H

pytestmark = pytest.mark.gpu


def _graph(blest, rp, col, **opts):
    return blest.Graph(rp, col, **{"async": 1}, **opts)


@pytest.mark.parametrize("opt", [dict(update_scheme=0), dict(update_scheme=1), dict(persistent=0, update_scheme=0)])
def test_single_source_calls_back_to_back(opt):
    import torch
    from paper_2606_05081_amd import blest
    rp, col = inputs.rmat_graph(12, 31)
    srcs = inputs.sources(rp, 6, seed=32)
    with _graph(blest, rp, col, **opt) as g:
        outs = [torch.empty(g.n, dtype=torch.int32, device="cuda") for _ in srcs]
        for rep in range(2):
            for s, o in zip(srcs, outs):
                g.bfs(int(s), o)
            g.sync()
            last = oracle.bfs(rp, col, int(srcs[-1]))
            assert len(g.level_stats()) == last.max() + 1
            for s, o in zip(srcs, outs):
                assert np.array_equal(o.cpu().numpy(), oracle.bfs(rp, col, int(s)))


@pytest.mark.parametrize("graph_mode", [0, 1])
def test_multi_source_calls_back_to_back(graph_mode):
    import torch
    from paper_2606_05081_amd import blest
    rp, col = inputs.rmat_graph(12, 33)
    every = inputs.sources(rp, 1200, seed=34, distinct=False)
    parts = [every[:64], every[64:300], every[300:1200], every[5:6]]  # in the arguments, and copied
    with _graph(blest, rp, col, msbfs_width=128, msbfs_graph=graph_mode) as g:
        outs = [torch.empty((len(p), g.n), dtype=torch.int16, device="cuda") for p in parts]
        cc = []
        for p, o in zip(parts, outs):
            mine = p.copy()
            g.msbfs(mine, o)
            mine[:] = -1  # the caller's list is its own again once the call returns
            cc.append(g.closeness(p))
        level = g.bfs(int(every[0]))
        g.sync()
        assert np.array_equal(level.cpu().numpy(), oracle.bfs(rp, col, int(every[0])))
        for p, o, (s, r, c) in zip(parts, outs, cc):
            assert np.array_equal(o.cpu().numpy(), oracle.msbfs16(rp, col, p))
            osum, oreach, occ = oracle.closeness(rp, col, p)
            assert np.array_equal(s.cpu().numpy(), osum) and np.array_equal(r.cpu().numpy(), oreach)
            assert np.array_equal(c.cpu().numpy(), occ)


def test_an_error_is_kept_until_the_sync():
    """A distance beyond int16 in the first call: the sync reports it although
    good calls follow, and the graph is good again after it."""
    import torch
    from paper_2606_05081_amd import blest
    rp, col = H.path(33000)
    with _graph(blest, rp, col) as g:
        good = g.bfs(7)
        g.sync()
        assert np.array_equal(good.cpu().numpy(), oracle.bfs(rp, col, 7))
        bad = torch.empty((2, g.n), dtype=torch.int16, device="cuda")
        for follow in (0, 2):
            g.msbfs([0, 5], bad)
            for _ in range(follow):
                g.bfs(16000)
                g.closeness([16000])
            with pytest.raises(blest.BlestError) as ei:
                g.sync()
            assert ei.value.status == blest.Status.OVERFLOW
            g.sync()  # reported once
            lev = g.msbfs([16000])
            one = g.bfs(3)
            g.sync()
            assert np.array_equal(lev.cpu().numpy(), oracle.msbfs16(rp, col, [16000]))
            assert np.array_equal(one.cpu().numpy(), oracle.bfs(rp, col, 3))
