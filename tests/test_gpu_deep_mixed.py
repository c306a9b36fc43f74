"""Deep claim-word searches on different graphs together, past the list length
where a launch expands one level only (a step of the whole grid): rows of four
entries throughout, and of four and eight mixed.  Bit for bit the oracle's."""
import numpy as np
import pytest

import graphgen
import oracle
from gpu_common import need_gpu, say

pytestmark = pytest.mark.gpu


def _matchings(n, k, seed):
    """k random perfect matchings: every degree at most k, levels that double."""
    rng = np.random.default_rng(seed)
    p = [rng.permutation(n) for _ in range(k)]
    return graphgen.from_edges(n, np.concatenate([x[0:n - 1:2] for x in p]), np.concatenate([x[1:n:2] for x in p]))


MIXES = {
    "rows of 4": lambda: [_matchings(600001, 3, 1), graphgen.grid(150, 0.9, 2), graphgen.path_graph(700),
                          _matchings(300000, 4, 3)],
    "rows of 4 and 8": lambda: [_matchings(200000, 8, 4), _matchings(600001, 3, 5), graphgen.star_graph(9),
                                graphgen.binary_tree(5000)],
    "one of them again": lambda: [_matchings(400000, 8, 6), graphgen.path_graph(3)],
}


@pytest.mark.parametrize("name", list(MIXES))
def test_mixed_wide_lists(name):
    import torch
    P = need_gpu()
    gs = MIXES[name]()
    if name == "one of them again":
        gs = [gs[0], gs[1], gs[0]]
    Gs = [P.Graph.from_graphgen(g) for g in gs]
    src = [g.n // 2 for g in gs]
    say(f"[deep mixed] {name}")
    info = {}
    lv, pa = P.bfs_batch(Gs, src, info=info)
    torch.cuda.synchronize()
    assert info["push_used"] == "claim"
    want = [oracle.bfs_graph(g, s) for g, s in zip(gs, src)]
    for q, (wl, wp) in enumerate(want):
        assert np.array_equal(lv[q].cpu().numpy(), wl) and np.array_equal(pa[q].cpu().numpy(), wp), (name, q)
    # a level of more than 2,048 waves' 64 columns over the queries together
    joint = np.zeros(max(int(w[0].max()) for w in want) + 1, np.int64)
    for wl, _ in want:
        joint += np.bincount(wl[wl >= 0], minlength=joint.size)
    assert joint.max() > 2048 * 64
