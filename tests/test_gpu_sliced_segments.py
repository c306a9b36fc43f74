"""The sliced push's segments (a wave's share of the bitmap, 2 to 64 words, by
the graph's size and slices) and the automatic choice of the form at its
bounds.  Bit for bit the oracle's."""
import numpy as np
import pytest

import graphgen
from gpu_common import assert_same, need_gpu, run_gpu, say

pytestmark = pytest.mark.gpu


def _mesh(side):
    """A three-dimensional mesh of 26 neighbours."""
    v = np.arange(side ** 3).reshape(side, side, side)
    src, dst = [], []
    for d in np.ndindex(3, 3, 3):
        if d > (1, 1, 1):
            a = tuple(slice(max(0, 1 - x), side - max(0, x - 1)) for x in d)
            b = tuple(slice(max(0, x - 1), side - max(0, 1 - x)) for x in d)
            src.append(v[a].ravel())
            dst.append(v[b].ravel())
    return graphgen.from_edges(side ** 3, np.concatenate(src), np.concatenate(dst))


def _rmat(n, seed, directed=False, per=4):
    """R-MAT edges folded onto n vertices."""
    rng = np.random.default_rng(seed)
    g = graphgen.rmat(max(6, (n - 1).bit_length()), per, seed, directed=directed)
    s = np.repeat(np.arange(g.n), np.diff(g.ptr)) % n
    return graphgen.from_edges(n, s, g.idx % n, directed=directed)


@pytest.mark.parametrize("n, directed", [(40, False), (2049, True), (140001, False), (270001, True),
                                         (1050001, False), (1100033, True), (2200001, False)])
def test_segments(n, directed):
    P = need_gpu()
    g = _rmat(n, n, directed)
    G = P.Graph.from_graphgen(g)
    for words in (32768, 4096) if n <= 500000 else (32768,):
        G.set_slice_words(words)
        for s in graphgen.pick_sources(g, 2, 7):
            for kw in (dict(), dict(loop="graph", levels_per_sync=3)):
                say(f"[segments] n={n} words={words} s={s} {kw}")
                assert_same(g, int(s), run_gpu(P, G, int(s), push_impl="sliced", **kw), f"segments/{n}/{s}")


@pytest.mark.parametrize("name, build, want", [
    ("skewed at the bound", lambda: _rmat(3 << 14, 3, per=16), "sliced"),
    ("skewed below it", lambda: _rmat((3 << 14) - 1, 3, per=16), "list"),
    ("even, wide levels", lambda: graphgen.erdos_renyi(1 << 18, 14, 4), "sliced"),
    ("even, few entries", lambda: graphgen.erdos_renyi(1 << 18, 9, 5), "list"),
    ("even, narrow levels", lambda: _mesh(65), "list"),
])
def test_choice(name, build, want):
    P = need_gpu()
    g = build()
    G = P.Graph.from_graphgen(g)
    s = int(graphgen.pick_sources(g, 1, 11)[0])
    info = {}
    say(f"[choice] {name} s={s}")
    assert_same(g, s, run_gpu(P, G, s, info=info), name)
    assert info["push_used"] == want
    # counted searches and several roots stay with the list form below 2^17
    # vertices and on even degrees
    info = {}
    assert_same(g, s, run_gpu(P, G, s, count_atomics=1, info=info), name)
    assert info["push_used"] == "list" and info["atomics"] > 0
    info = {}
    P.bfs_roots(G, [s, (s + 1) % g.n], info=info)
    assert info["push_used"] == "list"
