"""Each switch network keeps its own confidence floor, whichever is installed
last: a floor of 1 makes every level of its calls fall back, one of 0.34 (just
above the smallest winning probability of three) none that is in range."""
import numpy as np
import pytest

from paper_2606_05081_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("single_first", [True, False])
@pytest.mark.parametrize("single,multi", [(1.0, 0.34), (0.34, 1.0)])
def test_floor_of_each_network(single, multi, single_first):
    from paper_2606_05081_amd import blest, switch
    rp, col = inputs.rmat_graph(13, 71)
    srcs = inputs.sources(rp, 64, seed=72)
    # logits zero but for the biases: engine 2 with probability e / (e + 2), 0.58
    params = np.zeros(blest.MLP_NPARAMS, np.float32)
    params[-1] = 1.0
    std = np.full(12, 8.0, np.float32)
    with blest.Graph(rp, col, policy=int(blest.Policy.LEARNED)) as g:
        setters = [(g.set_switch_model, single), (g.set_ms_switch_model, multi)]
        for setter, floor in setters if single_first else setters[::-1]:
            setter(params, np.zeros(12, np.float32), std, floor)
        g.bfs(int(srcs[0]))
        fell = [r["mlp_fallback"] for r in g.level_stats()[:-1]]
        g.closeness(srcs)
        ms_fell = [r["mlp_fallback"] for r in g.ms_level_stats()]
    assert set(fell) == {int(single == 1.0)} and set(ms_fell) == {int(multi == 1.0)}
