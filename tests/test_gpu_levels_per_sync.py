"""levels_per_sync changes no result and refuses nothing, however many levels the
search has: graphs of one vertex and up, every variant and form of the push."""
import numpy as np
import pytest

import graphgen
from gpu_common import assert_same, need_gpu, run_gpu, say

pytestmark = pytest.mark.gpu

GRAPHS = {
    "n1": lambda: graphgen.from_edges(1, np.array([], int), np.array([], int)),
    "path5": lambda: graphgen.path_graph(5),
    "star40": lambda: graphgen.star_graph(40),
    "random": lambda: graphgen.erdos_renyi(900, 8, 3),
}


@pytest.mark.parametrize("name", list(GRAPHS))
def test_any_levels_per_sync(name):
    P = need_gpu()
    g = GRAPHS[name]()
    G = P.Graph.from_graphgen(g)
    runs = [dict(variant=v, loop=loop) for v in ("push", "pull", "bitmap", "heuristic", "short_circuit")
            for loop in ("host", "graph")]
    runs += [dict(push_impl=i) for i in ("list", "sliced", "claim")]
    for kw in runs:
        for per in (1, 2, 64, 4096):
            if per == 4096 and kw.get("loop") == "graph":
                continue                          # 4,097 launches a replay
            say(f"[levels_per_sync] {name} {kw} {per}")
            info = {}
            got = run_gpu(P, G, 0, levels_per_sync=per, info=info, **kw)
            assert_same(g, 0, got, f"{name} {kw} {per}")
            assert info["levels"] == int(got[0].max()) + 1
