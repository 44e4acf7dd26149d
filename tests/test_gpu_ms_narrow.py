"""Multi-source batches of fewer sources than their width: a vertex keeps only
the words that the sources need (1, 2, 4 or 8), at the counts where their number
changes, every output and both launch forms, wider batches of other calls on the
same graph in between. All outputs have one correct value: array equality."""
import numpy as np
import pytest

import oracle
from paper_2606_05081_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("graph_mode", [0, 1])
@pytest.mark.parametrize("sigma", [8, 16])
def test_counts_below_the_width(sigma, graph_mode):
    import torch
    from paper_2606_05081_amd import blest
    rp, col = inputs.rmat_graph(11, 77)
    n = rp.size - 1
    every = inputs.sources(rp, 600, seed=78, distinct=False)
    ref, (osum, oreach, occ) = oracle.msbfs16(rp, col, every), oracle.closeness(rp, col, every)
    g = blest.Graph(rp, col, sigma=sigma, msbfs_width=512, msbfs_graph=graph_mode)
    for k in (1, 63, 64, 65, 600, 128, 129, 256, 257, 512, 513, 3):
        srcs = every[:k]
        assert np.array_equal(g.msbfs(srcs).cpu().numpy(), ref[:k]), k
        assert np.array_equal(g.msbfs_batched(srcs, [256, 64, 512]).cpu().numpy(), ref[:k]), k
        out = torch.full((k, n), 7, dtype=torch.int16, device="cuda")
        assert np.array_equal(g.msbfs_noalloc(srcs, out).cpu().numpy(), ref[:k]), k
        s, r, c = g.closeness(srcs)
        assert np.array_equal(s.cpu().numpy(), osum[:k]) and np.array_equal(r.cpu().numpy(), oreach[:k]), k
        assert np.array_equal(c.cpu().numpy(), occ[:k]), k
        assert np.array_equal(g.far(srcs).cpu().numpy(), oracle.far(rp, col, srcs)), k
    g.close()
