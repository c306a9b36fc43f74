"""Sliced push on levels of few and of many vertices in one search: the bitmap words
that a wave takes at a time change from level to level (longer segments on thin
levels of large graphs), at sizes where they start, with a ragged last
segment and with several slices.  Bit for bit the oracle's."""
import numpy as np
import pytest

import graphgen
from gpu_common import assert_same, need_gpu, run_gpu, say

pytestmark = pytest.mark.gpu


def _tadpole(n, seed):
    """A random graph of degree 8 over two thirds of the vertices, a path over the rest."""
    rng = np.random.default_rng(seed)
    m = 2 * n // 3
    e = rng.integers(0, m, (2, 4 * m))
    path = np.arange(m - 1, n)
    p = rng.permutation(n)
    return graphgen.from_edges(n, p[np.concatenate([e[0], path[:-1]])], p[np.concatenate([e[1], path[1:]])])


def _short_tail(n, seed):
    """The same with a path of 60 and the other vertices alone."""
    rng = np.random.default_rng(seed)
    m = 2 * n // 3
    e = rng.integers(0, m, (2, 4 * m))
    path = np.arange(m - 1, m + 60)
    p = rng.permutation(n)
    return graphgen.from_edges(n, p[np.concatenate([e[0], path[:-1]])], p[np.concatenate([e[1], path[1:]])])


@pytest.mark.parametrize("n", [(1 << 18) - 1, 1 << 18, 400003, 1100003])
def test_thin_and_wide_levels(n):
    P = need_gpu()
    g = _short_tail(n, n)
    G = P.Graph.from_graphgen(g)
    far = int(np.argmax(run_gpu(P, G, int(np.argmax(g.out_degree())), push_impl="list")[0]))
    for s in (far, int(np.argmax(g.out_degree()))):
        for kw in (dict(), dict(loop="graph", levels_per_sync=5)):
            say(f"[thin levels] n={n} s={s} {kw}")
            assert_same(g, s, run_gpu(P, G, s, push_impl="sliced", **kw), f"thin/{n}/{s}")


def test_thin_levels_in_several_slices():
    P = need_gpu()
    g = _tadpole(300, 1)
    G = P.Graph.from_graphgen(g)
    G.set_slice_words(4)
    say("[thin levels] 300 vertices, 3 slices")
    assert_same(g, 7, run_gpu(P, G, 7, push_impl="sliced"), "thin/300")
    g = _short_tail(1 << 18, 9)
    G = P.Graph.from_graphgen(g)
    for words in (2048, 4096):
        G.set_slice_words(words)
        say(f"[thin levels] 2^18 vertices, slices of {words} words")
        assert_same(g, 11, run_gpu(P, G, 11, push_impl="sliced"), f"thin/2^18/{words}")
