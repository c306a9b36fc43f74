"""Multi-source pulls over several mask words (more than 64 sources): two, three,
four and five words, whole and ragged last ones, rows of every class (a lane per
row and word, a wave, chunks; one workgroup, so that the later chunks get a
launch of their own), with and without the degree-ordered copy, per-source and
vertex-major results.  Bit for bit the oracle's."""
import numpy as np
import pytest

import graphgen
from gpu_common import compare_all, need_gpu, oracle_all, say

pytestmark = pytest.mark.gpu


def _mixed_rows(directed):
    """Rows of 0 to 40 entries, some of a few hundred and a few of thousands."""
    rng = np.random.default_rng(11)
    n = 3001
    deg = np.concatenate([rng.integers(0, 40, n - 40), rng.integers(60, 500, 30), rng.integers(1200, 2900, 10)])
    rng.shuffle(deg)
    src = np.repeat(np.arange(n), deg)
    return graphgen.from_edges(n, src, rng.integers(0, n, len(src)), directed=directed)


@pytest.mark.parametrize("nq", [65, 128, 150, 256, 300])
@pytest.mark.parametrize("directed", [False, True])
def test_words(nq, directed):
    P = need_gpu()
    g = _mixed_rows(directed)
    src = [int(s) for s in np.random.default_rng(nq).integers(0, g.n, nq)]
    want = oracle_all(g, src)
    for order in (False, True):
        G = P.Graph.from_graphgen(g, ms_degree_order=order)
        for kw in (dict(variant="pull"), dict(variant="pull", grid_blocks=1), dict(variant="heuristic")):
            say(f"[words] nq={nq} directed={directed} order={order} {kw}")
            lv, pa = P.bfs_batch(G, src, **kw)
            compare_all(want, src, lambda q: (lv[q].cpu().numpy(), pa[q].cpu().numpy()), "words batch")
            vl, vp = P.bfs_batch_vm(G, src, **kw)
            vl, vp = vl.cpu().numpy(), vp.cpu().numpy()
            compare_all(want, src, lambda q: (vl[:, q], vp[:, q]), "words matrix")
            assert (vl[:, nq:] == -1).all() and (vp[:, nq:] == -1).all()
