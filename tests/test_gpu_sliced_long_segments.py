"""Sliced push where its longer segments on thin levels begin, 3 x 2^17 vertices: the
sizes beside it, and past it in several slices with a ragged last segment, on searches
with thin levels and wide ones.  Bit for bit the oracle's."""
import numpy as np
import pytest

from gpu_common import assert_same, need_gpu, run_gpu, say
from test_gpu_sliced_thin import _short_tail

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,words", [(3 * (1 << 17) - 1, 0), (3 * (1 << 17), 0), (3 * (1 << 17) + 33, 4096),
                                     (3 * (1 << 17) + 33, 6144)])
def test_segments(n, words):
    P = need_gpu()
    g = _short_tail(n, n)
    G = P.Graph.from_graphgen(g)
    if words:
        G.set_slice_words(words)
    hub = int(np.argmax(g.out_degree()))
    far = int(np.argmax(run_gpu(P, G, hub, push_impl="list")[0]))
    for s in (far, hub):
        say(f"[segments] n={n} words={words} s={s}")
        assert_same(g, s, run_gpu(P, G, s, push_impl="sliced"), f"segments/{n}/{words}/{s}")
