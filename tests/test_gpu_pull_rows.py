"""Bottom-up steps over rows of every length round the blocks of four columns
that a lane reads, with the only frontier neighbour at every position of the
row. Levels are integers: array equality."""
import numpy as np
import pytest

import oracle
from paper_2606_05081_amd import inputs

pytestmark = pytest.mark.gpu

LENGTHS = [1, 3, 4, 5, 7, 8, 9, 12, 15, 16, 17, 31, 32, 33, 48, 80]


def _one_hit_rows():
    """Vertices whose rows hold p vertices below f, f itself and the rest above
    it, for every length and p; f is the only neighbour of the source."""
    pool = max(LENGTHS)
    f, src, first = pool, 2 * pool + 1, 2 * pool + 2
    us, vs, at = [np.array([src])], [np.array([f])], first
    for length in LENGTHS:
        for p in range(length):
            row = np.concatenate([np.arange(p), [f], f + 1 + np.arange(length - 1 - p)])
            us.append(np.full(row.size, at))
            vs.append(row)
            at += 1
    return at, np.concatenate(us), np.concatenate(vs), src


@pytest.mark.parametrize("scheme", [0, 1])
@pytest.mark.parametrize("sigma", [8, 16, 32])
def test_hit_at_every_position(sigma, scheme):
    from paper_2606_05081_amd import blest
    n, us, vs, src = _one_hit_rows()
    rows = n - src - 1
    for repeat in (1, 9):  # one chunk of vertices a wave, and several
        u = np.concatenate([np.where(us > src, us + i * rows, us) for i in range(repeat)])
        rp, col = inputs.from_pairs(n + (repeat - 1) * rows, u, np.concatenate([vs] * repeat))
        ref = oracle.bfs(rp, col, src)
        assert (ref[src + 1:] == 2).all()
        g = blest.Graph(rp, col, reorder=0, sigma=sigma, update_scheme=scheme)
        g.set_policy(blest.Policy.BOTTOM_UP)
        assert np.array_equal(g.bfs(src).cpu().numpy(), ref)
        g.close()
