"""Queries on different graphs packed into one block-diagonal matrix: tiles that
one query fills, that several share, that hold many tiny queries, queries
without entries, the last tile's padding.  Bit for bit the oracle's."""
import numpy as np
import pytest

import graphgen
from gpu_common import assert_same, need_gpu, say

pytestmark = pytest.mark.gpu


def _empty(n):
    return graphgen.from_edges(n, np.zeros(0, np.int64), np.zeros(0, np.int64))


CASES = {
    "one tile each": lambda: [graphgen.erdos_renyi(512, 8, k) for k in range(5)],
    "tiny": lambda: [graphgen.star_graph(11 + k % 7) for k in range(700)],
    "large and small": lambda: [graphgen.erdos_renyi(n, 12, n) for n in (30011, 17, 1024, 5, 40000, 2049)],
    "no entries": lambda: [_empty(3), graphgen.erdos_renyi(3000, 10, 3), _empty(1), _empty(2000),
                           graphgen.star_graph(300), _empty(7)],
    "nothing at all": lambda: [_empty(5), _empty(1500)],
}


@pytest.mark.parametrize("name", list(CASES))
def test_pack(name):
    P = need_gpu()
    import torch
    gs = CASES[name]()
    Gs = [P.Graph.from_graphgen(g) for g in gs]
    src = [(7 * k) % g.n for k, g in enumerate(gs)]
    say(f"[pack] {name}")
    lv, pa = P.bfs_batch(Gs, src, push_impl="list")
    torch.cuda.synchronize()
    for k, g in enumerate(gs):
        assert_same(g, src[k], (lv[k].cpu().numpy(), pa[k].cpu().numpy()), f"pack/{name}/{k}")
