"""The multi-source gather step at the sizes where its row classes, lane groups
and front-bit words change: rows one below, at and one above every degree
bound, vertex counts that are no multiple of a wave's rows, every batch width
and slice-set width, levels kept as planes and written directly. Levels, sums
and distances are integers: array equality with the oracle."""
import numpy as np
import pytest

import oracle
from paper_2606_05081_amd import inputs

pytestmark = pytest.mark.gpu

# degree bounds of the row classes: 32, 256 and 4096
DEGREES = [1, 7, 8, 9, 31, 32, 33, 64, 65, 127, 128, 129, 255, 256, 257, 511, 4095, 4096, 4097, 9000]


def _hubs(extra):
    """Hubs of the degrees above over a common pool of leaves (plus an arc to
    the next hub), a path of isolated-from-the-rest vertices, `extra` more."""
    leaves = max(DEGREES)
    us, vs = [], []
    for i, d in enumerate(DEGREES):
        link = 1 if i + 1 < len(DEGREES) else 0
        inn = 1 if i else 0
        pool = (np.arange(max(d - link - inn, 0)) * 7919 + 31 * i) % leaves
        us.append(np.full(pool.size + link, leaves + i))
        vs.append(np.concatenate([pool, np.full(link, leaves + i + 1)]))
    base = leaves + len(DEGREES)
    us.append(np.arange(base, base + 20))
    vs.append(np.arange(base + 1, base + 21))
    n = base + 21 + extra
    return inputs.from_pairs(n, np.concatenate(us), np.concatenate(vs))


@pytest.mark.parametrize("sigma", [8, 16, 32])
@pytest.mark.parametrize("extra", [0, 5])
def test_gather_row_classes(sigma, extra):
    import torch
    from paper_2606_05081_amd import blest
    rp, col = _hubs(extra)
    n = rp.size - 1
    deg = np.diff(rp)
    assert set(DEGREES[5:]) <= set(deg.tolist())  # every bound is present
    srcs = np.concatenate([np.arange(n - 30, n), inputs.sources(rp, 70, seed=5)]).astype(np.int32)
    ref = oracle.msbfs16(rp, col, srcs)
    osum, oreach, occ = oracle.closeness(rp, col, srcs)
    ofar = oracle.far(rp, col, srcs)
    for width in (64, 128, 256, 512):
        g = blest.Graph(rp, col, sigma=sigma, msbfs_width=width)
        for pol in ("BVSS", "BOTTOM_UP", "HEURISTIC"):
            g.set_policy(getattr(blest.Policy, pol), 10.0, 3)
            assert np.array_equal(g.msbfs(srcs).cpu().numpy(), ref), (width, pol)
            out = torch.empty((srcs.size, n), dtype=torch.int16, device="cuda")
            assert np.array_equal(g.msbfs_noalloc(srcs, out).cpu().numpy(), ref), (width, pol)
            s, r, c = g.closeness(srcs)
            assert np.array_equal(s.cpu().numpy(), osum) and np.array_equal(r.cpu().numpy(), oreach)
            assert np.array_equal(c.cpu().numpy(), occ)
            assert np.array_equal(g.far(srcs).cpu().numpy(), ofar), (width, pol)
        g.close()


@pytest.mark.parametrize("length,planes", [(8, 3), (17, 5), (300, 9)])
def test_level_planes(length, planes):
    """Levels of 4, 8 and 15 planes' worth (a path as long as the deepest
    level), odd and even vertex counts, ragged source counts."""
    from paper_2606_05081_amd import blest
    for n in (length, length + 1):
        rp, col = inputs.from_pairs(n, np.arange(n - 1), np.arange(1, n))
        g = blest.Graph(rp, col)
        for k in (1, 2, 31, 32, 33, 63, 65, 129):
            srcs = (np.arange(k) * 5 % n).astype(np.int32)
            srcs[0] = 0
            ref = oracle.msbfs16(rp, col, srcs)
            assert int(ref.max()).bit_length() in (planes, planes + 1)
            for widths in ([64], [512]):
                assert np.array_equal(g.msbfs_batched(srcs, widths).cpu().numpy(), ref), (n, k, widths)
        g.close()
