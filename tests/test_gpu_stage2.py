"""Stage 2 of the lazy scheme at the sizes where its windows change: one slice
set per thread up to two windows a workgroup, four beyond; a last set that is
not full, a last window that is not full, rows on both sides of a push chunk,
input order kept or not, and the panel step's own Stage 2. Levels are integers
with one correct value, so every comparison is array equality."""
import numpy as np
import pytest

import oracle
from paper_2606_05081_amd import inputs
from tests import helpers as H
from tests.test_gpu_bfs import run_all_policies

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def blest():
    import torch
    from paper_2606_05081_amd import blest as b
    assert torch.cuda.is_available()
    b.lib()
    return b


def sparse(n, m, seed):
    """A path through every vertex's neighbourhood (so all are reached within
    few levels) plus m random edges and two hubs."""
    rng = np.random.default_rng(seed)
    u = np.concatenate([rng.integers(0, n, m), np.zeros(n // 16, np.int64), np.full(n // 64, n - 1)])
    v = np.concatenate([rng.integers(0, n, m), rng.integers(0, n, n // 16), rng.integers(0, n, n // 64)])
    keep = u != v
    return inputs.from_pairs(n, u[keep].astype(np.int32), v[keep].astype(np.int32))


# sets per window: 256 x 256 threads = 65,536 sets of 8; twice that is the
# line between one and four sets per thread at block size 256
@pytest.mark.parametrize("n", [1, 7, 9, 511, 513, 4097, 2 * 65536 * 8, 2 * 65536 * 8 + 1, 2 * 65536 * 8 + 4100])
@pytest.mark.parametrize("opt", [dict(block_size=256), dict(block_size=256, reorder=0, panel=0),
                                 dict(block_size=256, stage2_count_first=2)])
def test_lazy_windows(blest, n, opt):
    if n < 16:
        rp, col = H.path(n) if n > 1 else inputs.from_pairs(1, np.zeros(0, np.int32), np.zeros(0, np.int32))
    else:
        rp, col = sparse(n, 4 * n, 5 + n % 97)
    g = blest.Graph(rp, col, update_scheme=blest.Update.LAZY, blocks_per_cu=1, **opt)
    for src in sorted({0, n // 2}):
        ref = oracle.bfs(rp, col, src)
        run_all_policies(blest, g, src, ref, seeds=(1,))
        assert [r["frontier"] for r in g.level_stats()] == oracle.level_counts(ref).tolist()
    g.close()


@pytest.mark.parametrize("opt", [dict(sigma=16), dict(sigma=32), dict(sigma=16, reorder=0, persistent=0),
                                 dict(panel=2), dict(panel=2, panel_log2_rows=8), dict(stage2_count_first=0),
                                 dict(single_block=0, stage2_count_first=2)])
def test_lazy_options(blest, opt):
    for rp, col in (sparse(20011, 90000, 3), inputs.rmat_graph(13, 9)):
        g = blest.Graph(rp, col, update_scheme=blest.Update.LAZY, **opt)
        for src in (0, 77, rp.size - 2):
            ref = oracle.bfs(rp, col, src)
            run_all_policies(blest, g, src, ref, seeds=(2,))
            assert [r["frontier"] for r in g.level_stats()] == oracle.level_counts(ref).tolist()
        g.close()


@pytest.mark.parametrize("scheme", ["LAZY", "EAGER"])
@pytest.mark.parametrize("sigma", [8, 16, 32])
def test_bottom_up_row_lengths(blest, scheme, sigma):
    """Rows one below, at and one above every bound of the bottom-up scan (four
    columns a step, 16 by a lane, 32, 64 a wave step), whose only neighbour in
    the frontier is the first, the last, or one before the last."""
    lens = [1, 2, 3, 4, 5, 15, 16, 17, 31, 32, 33, 34, 47, 48, 79, 80, 81, 144, 145, 400]
    nrow = 3 * len(lens)
    leaves = max(lens)
    # ids: gate first, leaves, rows, gate last; every leaf belongs to a row only
    us, vs = [], []
    last = 1 + leaves + nrow
    for i in range(nrow):
        row, d, kind = 1 + leaves + i, lens[i // 3], i % 3
        gate = 0 if kind == 0 else last
        others = 1 + (np.arange(d - 1) * 7 + i) % leaves if d > 1 else np.zeros(0, np.int64)
        if kind == 2:
            others = np.concatenate([others[:-1], [last + 1]]) if d > 1 else others  # beyond the gate
        us.append(np.full(others.size + 1, row))
        vs.append(np.concatenate([others, [gate]]))
    src = last + 2
    us.append(np.array([src, src]))
    vs.append(np.array([0, last]))
    rp, col = inputs.from_pairs(src + 1, np.concatenate(us).astype(np.int32), np.concatenate(vs).astype(np.int32))
    g = blest.Graph(rp, col, sigma=sigma, reorder=0, update_scheme=getattr(blest.Update, scheme))
    for s in (src, 0, last, 1, 1 + leaves):
        ref = oracle.bfs(rp, col, s)
        run_all_policies(blest, g, s, ref, seeds=(1,))
        assert [r["frontier"] for r in g.level_stats()] == oracle.level_counts(ref).tolist()
    g.close()
