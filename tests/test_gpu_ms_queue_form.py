"""The queue form of multi-source levels (opts.ms_queue_form = 1) on the small
graphs that otherwise take the gather form at every level: every slice-set
width and slice format, both launch forms, every output, levels through planes
and written directly, directed graphs, and levels of both forms in turn. The
records tell which form each level took. All outputs have one correct value:
array equality with the oracle."""
import numpy as np
import pytest

import oracle
from paper_2606_05081_amd import inputs
from tests import helpers as H

pytestmark = pytest.mark.gpu


def _graph(name):
    if name == "rmat":
        return inputs.rmat_graph(12, 51)
    if name == "rmat_directed":
        return inputs.rmat_directed(12, 52)
    if name == "grid":
        return inputs.grid_graph(60, 3)
    if name == "path":
        return H.path(400)
    if name == "hubs":  # rows and slice sets of thousands of VSSs' worth of slices
        u = np.concatenate([np.full(9000, 3), np.full(4097, 9001), np.arange(9000, 9300)])
        v = np.concatenate([np.arange(4, 9004), np.arange(5, 4102), np.arange(9001, 9301)])
        keep = u != v
        return inputs.from_pairs(9310, u[keep], v[keep])
    return inputs.from_pairs(29, [0, 1, 2, 10, 11, 20], [1, 2, 3, 11, 12, 21])


def _check(g, srcs, ref, sums, far, widths=None):
    import torch
    got = g.msbfs(srcs) if widths is None else g.msbfs_batched(srcs, widths)
    assert np.array_equal(got.cpu().numpy(), ref)
    out = torch.full((len(srcs), g.n), 7, dtype=torch.int16, device="cuda")
    assert np.array_equal(g.msbfs_noalloc(srcs, out).cpu().numpy(), ref)
    s, r, c = g.closeness(srcs)
    assert np.array_equal(s.cpu().numpy(), sums[0]) and np.array_equal(r.cpu().numpy(), sums[1])
    assert np.array_equal(c.cpu().numpy(), sums[2])
    assert np.array_equal(g.far(srcs).cpu().numpy(), far)


@pytest.mark.parametrize("graph_mode", [0, 1])
@pytest.mark.parametrize("opt", [dict(), dict(wide_slices=1), dict(sigma=16), dict(sigma=32), dict(tau=64, reorder=0),
                                 dict(tau=256, reorder=0)])
@pytest.mark.parametrize("name", ["rmat", "rmat_directed", "grid", "path", "hubs", "disconnected"])
def test_queue_form_exact(name, opt, graph_mode):
    from paper_2606_05081_amd import blest
    rp, col = _graph(name)
    n = rp.size - 1
    directed = int(name == "rmat_directed")
    every = (np.arange(300) * 37 % n).astype(np.int32)
    for width, k in ((64, 130), (128, 128), (256, 200), (512, 300)):
        srcs = every[:k]
        ref, sums, far = oracle.msbfs16(rp, col, srcs), oracle.closeness(rp, col, srcs), oracle.far(rp, col, srcs)
        g = blest.Graph(rp, col, msbfs_width=width, msbfs_graph=graph_mode, ms_queue_form=1, directed=directed, **opt)
        for policy, forms in (("BVSS", {0}), ("RANDOM", {0, 1}), ("HEURISTIC", {0, 1})):
            g.set_policy(getattr(blest.Policy, policy), 10.0, 3)
            _check(g, srcs, ref, sums, far)
            recs = g.ms_level_stats()
            assert {r["gather"] for r in recs} <= forms, policy
            assert all(r["gather"] == (r["engine"] == int(blest.Engine.BOTTOM_UP)) for r in recs), policy
            if policy == "RANDOM" and len(recs) > 12:
                assert {r["gather"] for r in recs} == forms
        g.close()


def test_forms_of_the_full_method():
    """Without the option a small graph's levels are all gathered, whatever the
    engine, and the records say so; probe mode tells dense levels apart."""
    from paper_2606_05081_amd import blest
    rp, col = _graph("rmat")
    srcs = inputs.sources(rp, 100, seed=9)
    ref = oracle.msbfs16(rp, col, srcs)
    with blest.Graph(rp, col) as g:
        for policy in ("BVSS", "BOTTOM_UP"):
            g.set_policy(getattr(blest.Policy, policy))
            assert np.array_equal(g.msbfs(srcs).cpu().numpy(), ref)
            recs = g.ms_level_stats()
            assert all(r["gather"] == 1 for r in recs)
            assert {r["engine"] for r in recs} == {int(getattr(blest.Engine, policy))}
    for queue_form in (0, 1):
        with blest.Graph(rp, col, ms_queue_form=queue_form) as g:
            assert np.array_equal(g.msbfs_probe(srcs, [64]).cpu().numpy(), ref)
            recs = g.ms_level_stats()
            assert all(r["gather"] == 1 - queue_form and min(r["t_engine_us"]) > 0 for r in recs)
            same = [r["t_engine_us"][0] == r["t_engine_us"][1] for r in recs]
            assert all(same) if queue_form == 0 else not all(same)


def test_learned_policy_decides_queue_levels():
    """With the committed network on the queue form: exact, and both engines' levels occur."""
    from paper_2606_05081_amd import blest
    for rp, col in (inputs.grid_graph(60, 3), inputs.rmat_graph(12, 51)):
        srcs = inputs.sources(rp, 256, seed=10)
        ref, sums, far = oracle.msbfs16(rp, col, srcs), oracle.closeness(rp, col, srcs), oracle.far(rp, col, srcs)
        with blest.Graph(rp, col, ms_queue_form=1, msbfs_width=256, policy=int(blest.Policy.LEARNED)) as g:
            H.install_switch_models(g)
            _check(g, srcs, ref, sums, far)


@pytest.mark.parametrize("n", [907777, 1074561])
def test_queue_form_at_the_lds_limit(n):
    """Front bits in LDS or in memory beside queue levels, where the switch
    network's weights share the place of the queue form's tables or not."""
    from paper_2606_05081_amd import blest
    rng = np.random.default_rng(n)
    u, v = rng.integers(0, n, n), rng.integers(0, n, n)
    keep = u != v
    rp, col = inputs.from_pairs(n, u[keep].astype(np.int32), v[keep].astype(np.int32))
    srcs = inputs.sources(rp, 3, seed=5)
    ref = np.stack([oracle.bfs(rp, col, int(s)) for s in srcs])
    with blest.Graph(rp, col, reorder=0, msbfs_width=64, ms_queue_form=1) as g:
        H.install_switch_models(g)
        for pol in ("RANDOM", "LEARNED"):
            g.set_policy(getattr(blest.Policy, pol), 10.0, 2)
            assert np.array_equal(g.msbfs(srcs).cpu().numpy(), ref), pol
            recs = g.ms_level_stats()
            assert pol == "LEARNED" or {r["gather"] for r in recs} == {0, 1}
