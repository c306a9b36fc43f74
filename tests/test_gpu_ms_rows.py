"""Multi-source pulls over the degree-ordered copy's row chunks, whose bounds
follow the entries of their rows where the longest rows are many times a wave's
share: rows below and at the length that is split (511, 512 entries), rows that
fill a chunk alone and sixteen short ones, mixed in one graph, with all sources
joined, with some that never reach a row, undirected and directed, one mask word
and several.  Bit for bit the oracle's."""
import numpy as np
import pytest

import graphgen
from gpu_common import check_all, need_gpu, say

pytestmark = pytest.mark.gpu


def stepped(n, degrees, directed, seed):
    """Vertex i < len(degrees) with that many neighbours among the others; a few
    random edges between those, and some vertices without any."""
    rng = np.random.default_rng(seed)
    a, b = [], []
    for i, d in enumerate(degrees):
        x = len(degrees) + rng.permutation(n - len(degrees) - 50)[:d]
        a.append(np.full(d, i)), b.append(x)
    a.append(rng.integers(len(degrees), n - 50, n // 2)), b.append(rng.integers(len(degrees), n - 50, n // 2))
    a, b = np.concatenate(a), np.concatenate(b)
    if directed:        # in-lists as long as out-lists, of other vertices
        a, b = np.concatenate([a, rng.permutation(n)[:len(b)] if len(b) <= n else rng.integers(0, n, len(b))]), \
            np.concatenate([b, a])
    return graphgen.from_edges(n, a, b, directed=directed)


DEGREES = [700] * 3 + [512] * 2 + [511] * 37 + [300] * 30 + [128] * 50 + [40] * 20


@pytest.mark.parametrize("directed", [False, True])
@pytest.mark.parametrize("nq", [3, 64, 70, 200])
def test_row_chunks(directed, nq):
    import torch
    P = need_gpu()
    from paper_1906_03113_amd import selector
    g = stepped(6001, DEGREES, directed, 5)
    G = P.Graph.from_graphgen(g, ms_degree_order=True)
    net = selector.load_weights(selector.MS_WEIGHTS)
    src = [int(s) for s in np.random.default_rng(nq).integers(0, g.n, nq)]
    for variant, blocks in (("pull", 0), ("pull", 1), ("heuristic", 0), ("learned", 0)):
        kw = dict(selector=net) if variant == "learned" else {}
        say(f"[row chunks] directed={directed} nq={nq} {variant} blocks={blocks}")
        bl, bp = P.bfs_batch(G, src, variant=variant, grid_blocks=blocks, push_impl="list", **kw)
        torch.cuda.synchronize()
        check_all(g, src, lambda q: (bl[q].cpu().numpy(), bp[q].cpu().numpy()), f"batch {variant}")
        lv, pa = P.bfs_batch_vm(G, src, variant=variant, grid_blocks=blocks, **kw)
        torch.cuda.synchronize()
        lv, pa = lv.cpu().numpy(), pa.cpu().numpy()
        check_all(g, src, lambda q: (lv[:, q].copy(), pa[:, q].copy()), f"vm {variant}")
