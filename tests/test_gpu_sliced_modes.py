"""The sliced push's choice between its two kinds of level: few vertices with
many entries (hubs behind the root, one level later, on the way down), few with
few, many with many.  Bit for bit the oracle's, host and graph loop, one and
several slices."""
import numpy as np
import pytest

import graphgen
from gpu_common import assert_same, need_gpu, run_gpu, say

pytestmark = pytest.mark.gpu


def _hubs(n, depth, hubs, leaves, tail, seed):
    """A path of `depth` vertices, then `hubs` hubs with `leaves` random leaves
    each, then a path of `tail` vertices behind one leaf."""
    rng = np.random.default_rng(seed)
    src, dst = [np.arange(depth - 1)], [np.arange(1, depth)]
    h = depth + np.arange(hubs)
    src.append(np.full(hubs, depth - 1))
    dst.append(h)
    first = depth + hubs
    for v in h:
        src.append(np.full(leaves, v))
        dst.append(first + rng.integers(0, n - first - tail, leaves))
    t = n - tail + np.arange(tail)
    src.append(np.concatenate([[dst[-1][0]], t[:-1]]))
    dst.append(t)
    return graphgen.from_edges(n, np.concatenate(src), np.concatenate(dst))


CASES = {
    "hubs_at_once": lambda: _hubs(140001, 1, 30, 30000, 5, 1),
    "hubs_later": lambda: _hubs(140001, 4, 300, 4000, 9, 2),
    "one_hub": lambda: _hubs(131072, 2, 1, 120000, 3, 3),
    "rmat17": lambda: graphgen.rmat(17, 16, 4),
    "rmatd17": lambda: graphgen.rmat(17, 16, 5, directed=True),
}


@pytest.mark.parametrize("name", list(CASES))
def test_level_kinds(name):
    P = need_gpu()
    g = CASES[name]()
    G = P.Graph.from_graphgen(g)
    for words in (32768, 2048):                      # one slice; several
        G.set_slice_words(words)
        for s in (0, int(g.idx[0]), g.n - 1):
            for kw in (dict(), dict(loop="graph", levels_per_sync=3)):
                say(f"[sliced] {name} words={words} s={s} {kw}")
                assert_same(g, s, run_gpu(P, G, s, push_impl="sliced", **kw), f"sliced/{name}/{s}")
