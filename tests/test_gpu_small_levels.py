"""The list form's small levels, several to a launch by one workgroup: searches
that stay small, that cross the limit both ways (1,024 columns or entries), that
reach long columns, columns without entries, and the direction policies that
leave the push between them.  Bit for bit the oracle's, in the host and the
graph loop, and the same with every level its own launch (a traced run)."""
import numpy as np
import pytest

import graphgen
from gpu_common import assert_same, need_gpu, run_gpu, say

pytestmark = pytest.mark.gpu


def _bursts(widths, hub, seed):
    """Layers of the given widths, each vertex joined to a random one of the layer
    before; every `hub`-th layer's first vertex also joined to all of the next."""
    rng = np.random.default_rng(seed)
    off = np.concatenate([[0], np.cumsum(widths)])
    src, dst = [], []
    for k in range(len(widths) - 1):
        child = np.arange(off[k + 1], off[k + 2])
        src.append(off[k] + rng.integers(0, widths[k], len(child)))
        dst.append(child)
        if hub and k % hub == 0:
            src.append(np.full(len(child), off[k]))
            dst.append(child)
    return graphgen.from_edges(int(off[-1]), np.concatenate(src), np.concatenate(dst))


def _directed_sinks():
    """A root with 1,100 out-neighbours, all but one without out-entries."""
    src = np.concatenate([np.zeros(1100, int), [1, 2000, 2001]])
    dst = np.concatenate([np.arange(1, 1101), [2000, 2001, 2002]])
    return graphgen.from_edges(2100, src, dst, directed=True)


CASES = {
    "path900": lambda: graphgen.path_graph(900),
    "star1025": lambda: graphgen.star_graph(1026),
    "limit": lambda: _bursts([1, 3, 511, 512, 513, 1024, 1025, 7, 1, 1, 900, 2], 0, 1),
    "long_columns": lambda: _bursts([1, 40, 3, 700, 2, 5, 1500, 3, 9, 600, 1, 4], 2, 2),
    "er": lambda: graphgen.erdos_renyi(16384, 8, 3),
    "sinks": _directed_sinks,
    "rmatd": lambda: graphgen.rmat(12, 16, 4, directed=True),
}


@pytest.mark.parametrize("name", list(CASES))
def test_small_levels(name):
    P = need_gpu()
    from paper_1906_03113_amd import selector
    g = CASES[name]()
    G = P.Graph.from_graphgen(g)
    net = selector.load_weights()
    for s in (0, g.n // 2):
        for kw in (dict(variant="push", push_impl="list"), dict(variant="push", push_impl="list", loop="graph"),
                   dict(variant="heuristic"), dict(variant="learned", selector=net, loop="graph", levels_per_sync=3),
                   dict(variant="push", push_impl="list", heavy_degree=32, chunk_edges=64), dict(variant="bitmap")):
            say(f"[small] {name} s={s} {kw.get('variant')} {kw.get('loop', 'host')}")
            info, one = {}, {}
            got = run_gpu(P, G, s, info=info, **kw)
            assert_same(g, s, got, f"small/{name}/{s}")
            run_gpu(P, G, s, info=one, trace=True, **kw)
            assert info["levels"] == one["levels"] == int(got[0].max()) + 1
