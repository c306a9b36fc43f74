"""Multi-source pulls where rows of more than 16 entries begin: no such row, one of 17,
and a directed graph whose out-lists are short and whose in-lists are not, with and
without the degree order.  Bit for bit the oracle's."""
import numpy as np
import pytest

import graphgen
from gpu_common import check_all, need_gpu, say

pytestmark = pytest.mark.gpu


def _hub(n, degree, directed, seed):
    """A path (both ways) and one vertex with `degree` neighbours (in-neighbours where directed)."""
    rng = np.random.default_rng(seed)
    v = np.arange(n - 2)
    a, b = np.concatenate([v, rng.permutation(n - 1)[:degree]]), np.concatenate([v + 1, np.full(degree, n - 1)])
    if directed:
        a, b = np.concatenate([a, v + 1, [n - 1]]), np.concatenate([b, v, [0]])
    return graphgen.from_edges(n, a, b, directed=directed)


@pytest.mark.parametrize("degree,directed", [(15, False), (16, False), (17, False), (17, True), (600, True)])
@pytest.mark.parametrize("order", [False, True])
@pytest.mark.parametrize("nq", [5, 70, 200])
def test_rows_past_sixteen(degree, directed, order, nq):
    import torch
    P = need_gpu()
    g = _hub(901, degree, directed, degree)
    G = P.Graph.from_graphgen(g, ms_degree_order=order)
    src = [int(s) for s in np.random.default_rng(nq).integers(0, g.n, nq)]
    say(f"[wide edge] degree={degree} directed={directed} order={order} nq={nq}")
    bl, bp = P.bfs_batch(G, src, variant="pull", push_impl="list")
    torch.cuda.synchronize()
    check_all(g, src, lambda q: (bl[q].cpu().numpy(), bp[q].cpu().numpy()), "pull")
