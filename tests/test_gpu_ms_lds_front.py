"""Multi-source calls on both sides of two lines: front bits in LDS or read
from memory (1,074,560 vertices are the last that fit beside the kernel's other
LDS, 907,776 the last beside the switch network's weights too, which share the
place beyond), and source lists in the
kernel arguments (512 sources, 8 batches) or copied. Levels, sums and
distances are integers: array equality with the oracle."""
import numpy as np
import pytest

import oracle
from paper_2606_05081_amd import inputs
from tests import helpers as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [907776, 907777, 1074559, 1074560, 1074561, 1074600])
def test_front_bits_at_the_lds_limit(n):
    from paper_2606_05081_amd import blest
    rng = np.random.default_rng(n)
    u = np.concatenate([rng.integers(0, n, 2 * n), np.full(6000, n - 1), np.arange(n - 40, n - 1)])
    v = np.concatenate([rng.integers(0, n, 2 * n), rng.integers(0, n, 6000), np.arange(n - 39, n)])
    keep = u != v
    rp, col = inputs.from_pairs(n, u[keep].astype(np.int32), v[keep].astype(np.int32))
    srcs = np.array([0, n - 1, n // 2], dtype=np.int32)
    ref = np.stack([oracle.bfs(rp, col, int(s)) for s in srcs])
    g = blest.Graph(rp, col, reorder=0, msbfs_width=64)
    H.install_switch_models(g, multi=True)
    for pol in ("HEURISTIC", "LEARNED"):
        g.set_policy(getattr(blest.Policy, pol), 10.0, 1)
        assert np.array_equal(g.msbfs(srcs).cpu().numpy(), ref), pol
        s, r, _ = g.closeness(srcs)
        assert np.array_equal(s.cpu().numpy(), np.where(ref > 0, ref, 0).sum(axis=1))
        assert np.array_equal(r.cpu().numpy(), (ref >= 0).sum(axis=1))
    g.close()


@pytest.mark.parametrize("width", [64, 512])
@pytest.mark.parametrize("k", [1, 64, 65, 511, 512, 513])
def test_source_lists(k, width):
    from paper_2606_05081_amd import blest
    rp, col = inputs.rmat_graph(10, 7)
    srcs = (np.arange(k) * 37 % (rp.size - 1)).astype(np.int32)
    ref = oracle.msbfs16(rp, col, srcs)
    osum, oreach, _ = oracle.closeness(rp, col, srcs)
    for graph in (0, 1):
        g = blest.Graph(rp, col, msbfs_width=width, msbfs_graph=graph)
        assert np.array_equal(g.msbfs(srcs).cpu().numpy(), ref)
        s, r, _ = g.closeness(srcs)
        assert np.array_equal(s.cpu().numpy(), osum) and np.array_equal(r.cpu().numpy(), oreach)
        g.close()
