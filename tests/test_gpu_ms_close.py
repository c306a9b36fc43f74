"""Multi-source levels at the edges of how their ends are dealt out: one workgroup
and several (the last one to arrive closes a level, alone it does so at once),
fewer (row, word)s than a wave's 64 when the planes become levels, searches
around the 32 levels that the planes hold, one mask word and several.  Bit for
bit the oracle's."""
import numpy as np
import pytest

import graphgen
from gpu_common import check_all, need_gpu, say

pytestmark = pytest.mark.gpu

GRAPHS = {
    "n1": lambda: graphgen.from_edges(1, np.array([], int), np.array([], int)),
    "path5": lambda: graphgen.path_graph(5),
    "path33": lambda: graphgen.path_graph(33),
    "path257": lambda: graphgen.path_graph(257),
    "tree": lambda: graphgen.binary_tree(1030),
    "random": lambda: graphgen.erdos_renyi(2049, 9, 4),
    "skewed": lambda: graphgen.rmat(10, seed=3),
}


@pytest.mark.parametrize("name", list(GRAPHS))
@pytest.mark.parametrize("nq", [2, 67, 130])
def test_level_ends(name, nq):
    import torch
    P = need_gpu()
    from paper_1906_03113_amd import selector
    g = GRAPHS[name]()
    G = P.Graph.from_graphgen(g)
    net = selector.load_weights(selector.MS_WEIGHTS)
    src = [int(s) for s in np.random.default_rng(nq).integers(0, g.n, nq)]
    for variant, blocks in (("push", 1), ("push", 3), ("pull", 1), ("heuristic", 2), ("learned", 1), ("learned", 0)):
        kw = dict(selector=net) if variant == "learned" else {}
        say(f"[level ends] {name} nq={nq} {variant} blocks={blocks}")
        info = {}
        lv, pa = P.bfs_batch_vm(G, src, variant=variant, grid_blocks=blocks, info=info, **kw)
        torch.cuda.synchronize()
        lv, pa = lv.cpu().numpy(), pa.cpu().numpy()
        check_all(g, src, lambda q: (lv[:, q].copy(), pa[:, q].copy()), f"vm {name} {variant}")
        assert (lv[:, nq:] == -1).all() and (pa[:, nq:] == -1).all()
        assert info["levels"] == int(lv.max()) + 1
        bl, bp = P.bfs_batch(G, src, variant=variant, grid_blocks=blocks, push_impl="list", **kw)
        torch.cuda.synchronize()
        check_all(g, src, lambda q: (bl[q].cpu().numpy(), bp[q].cpu().numpy()), f"batch {name} {variant}")
