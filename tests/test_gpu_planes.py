"""Multi-source levels as bit planes: searches that end on either side of a new
plane (levels 7 / 8, 15 / 16) and of the last one (31 / 32, where the planes
become staged levels), per-source and vertex-major results, one and several
words, with the degree-ordered copy and without, and the timed profile of every
level.  Bit for bit the oracle's."""
import numpy as np
import pytest

import graphgen
from gpu_common import compare_all, need_gpu, oracle_all, say

pytestmark = pytest.mark.gpu


def _deep(depth, seed):
    """A random core with a tail of `depth` vertices (and a hub: not thin)."""
    rng = np.random.default_rng(seed)
    n = 400
    src, dst = rng.integers(0, n, 1500), rng.integers(0, n, 1500)
    tail = n + np.arange(depth)
    return graphgen.from_edges(n + depth, np.concatenate([src, [0], tail[:-1]]), np.concatenate([dst, [n], tail[1:]]))


@pytest.mark.parametrize("depth", [1, 3, 11, 26, 27, 28, 29, 43, 70])
def test_planes(depth):
    P = need_gpu()
    g = _deep(depth, depth)
    for nq in (3, 64, 70):
        src = [int(s) for s in np.random.default_rng(nq).integers(0, g.n, nq)]
        want = oracle_all(g, src)
        for order in (False, True):
            G = P.Graph.from_graphgen(g, ms_degree_order=order)
            for kw in (dict(variant="push"), dict(variant="pull"), dict(variant="heuristic", ms_ranges=3)):
                say(f"[planes] depth={depth} nq={nq} order={order} {kw}")
                info = {}
                lv, pa = P.bfs_batch(G, src, info=info, **kw)
                compare_all(want, src, lambda q: (lv[q].cpu().numpy(), pa[q].cpu().numpy()), "planes batch")
                assert info["levels"] == max(int(w[0].max()) for w in want) + 1
                vl, vp = P.bfs_batch_vm(G, src, **kw)
                vl, vp = vl.cpu().numpy(), vp.cpu().numpy()
                compare_all(want, src, lambda q: (vl[:, q], vp[:, q]), "planes matrix")
                assert (vl[:, nq:] == -1).all() and (vp[:, nq:] == -1).all()


@pytest.mark.parametrize("depth", [5, 40])
def test_planes_profile(depth):
    from paper_1906_03113_amd import selector
    P = need_gpu()
    g = _deep(depth, depth)
    G = P.Graph.from_graphgen(g)
    src = [int(s) for s in np.random.default_rng(1).integers(0, g.n, 20)]
    say(f"[planes] profile depth={depth}")
    import torch
    out = [torch.empty((g.n, 64), dtype=torch.int32, device="cuda") for _ in range(2)]
    selector.ms_profile(G, src, out=out)
    want = oracle_all(g, src)
    lv, pa = (x.cpu().numpy() for x in out)
    compare_all(want, src, lambda q: (lv[:, q], pa[:, q]), "planes profile")
