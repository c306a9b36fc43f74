"""The claim-word push on thin graphs, where waves carry their shares on for
many levels per launch: frontiers that grow past one step of the grid, rows of
one to eight entries, one vertex, deep paths, several queries on one graph and
on graphs of both row widths.  Bit for bit the oracle's."""
import ctypes

import numpy as np
import pytest

import graphgen
import oracle
from gpu_common import assert_same, check_all, need_gpu, run_gpu, say

pytestmark = pytest.mark.gpu


def _matchings(n, k, seed):
    """k random perfect matchings: every degree at most k, levels that double."""
    rng = np.random.default_rng(seed)
    p = [rng.permutation(n) for _ in range(k)]
    return graphgen.from_edges(n, np.concatenate([x[0:n - 1:2] for x in p]), np.concatenate([x[1:n:2] for x in p]))


def _relabelled(g, seed):
    """The same graph under a random labelling: no order between neighbours."""
    p = np.random.default_rng(seed).permutation(g.n)
    rows = np.repeat(np.arange(g.n), g.out_degree())
    return graphgen.from_edges(g.n, p[rows], p[g.idx])


CASES = {
    "n1": lambda: graphgen.from_edges(1, np.array([], int), np.array([], int)),
    "n2": lambda: graphgen.path_graph(2),
    "path700": lambda: graphgen.path_graph(700),
    "cycle129": lambda: graphgen.cycle_graph(129),
    "star8": lambda: graphgen.star_graph(9),                    # a row of eight entries
    "grid_ragged": lambda: graphgen.grid(203, 0.9, 5, height=97),
    "grid_shuffled": lambda: _relabelled(graphgen.grid(180, 0.9, 6), 7),
    "tree": lambda: graphgen.binary_tree(70001),
    "matchings3": lambda: _matchings(600001, 3, 8),             # lists past one step of the grid
    "matchings8": lambda: _matchings(200000, 8, 9),
}


@pytest.mark.parametrize("name", list(CASES))
def test_deep_levels(name):
    P = need_gpu()
    g = CASES[name]()
    assert g.n == 1 or g.out_degree().max() <= 8
    G = P.Graph.from_graphgen(g)
    for s in sorted({0, g.n // 2, g.n - 1}):
        say(f"[deep] {name} s={s}")
        info = {}
        got = run_gpu(P, G, s, info=info)
        assert info["push_used"] == "claim"
        assert_same(g, s, got, f"deep/{name}/{s}")
        assert info["levels"] == int(got[0].max()) + 1
    src = [0, g.n - 1, g.n // 3, 0]
    say(f"[deep] {name} batch")
    lv, pa = P.bfs_batch(G, src, push_impl="claim")
    check_all(g, src, lambda q: (lv[q].cpu().numpy(), pa[q].cpu().numpy()), f"deep batch/{name}")


def test_deep_on_graphs_of_both_row_widths():
    P = need_gpu()
    gs = [graphgen.grid(90, 0.9, 1), CASES["star8"](), graphgen.path_graph(333), _matchings(5000, 7, 2)]
    Gs = [P.Graph.from_graphgen(g) for g in gs]
    src = [17, 3, 200, 4999]
    say("[deep] mixed widths")
    info = {}
    lv, pa = P.bfs_batch(Gs, src, info=info)
    assert info["push_used"] == "claim"
    for q, g in enumerate(gs):
        wl, wp = oracle.bfs_graph(g, src[q])
        assert np.array_equal(lv[q].cpu().numpy(), wl) and np.array_equal(pa[q].cpu().numpy(), wp), q


@pytest.mark.parametrize("variant,nq", [("learned", 2), ("heuristic", 21), ("push", 64), ("learned", 130)])
def test_deep_batch_policies(variant, nq):
    """Many sources on a slowly growing thin graph: one group of claim-word
    searches or several, in a workspace of exactly the size asked for and in a
    smaller one; with a trace the multi-source levels run.  All the oracle's
    results and one level count."""
    import torch
    P = need_gpu()
    g = CASES["grid_ragged"]()
    G = P.Graph.from_graphgen(g)
    src = [int(s) for s in np.random.default_rng(nq).integers(0, g.n, nq)]
    counts = set()
    L = P._lib.lib()
    small = max(G.workspace_size(1), g.n * 600 * ((nq + 63) // 64) + 65536)     # the multi-source masks
    for trace, size in ((False, G.workspace_size(nq)), (False, small), (True, G.workspace_size(nq))):
        say(f"[deep] {variant} nq={nq} trace={trace} workspace={size}")
        ws = P.Workspace(size)
        lv = [torch.empty(g.n, dtype=torch.int32, device="cuda") for _ in src]
        pa = [torch.empty_like(x) for x in lv]
        opt, recs = P.make_options(variant, trace_capacity=(g.n + 2) if trace else 0)
        ptrs = lambda a: (ctypes.c_void_p * nq)(*[x.data_ptr() for x in a])
        P._lib.check(L.bfs_run_batch(nq, (ctypes.c_void_p * nq)(*[G.handle] * nq), (ctypes.c_int32 * nq)(*src),
                                     ptrs(lv), ptrs(pa), ctypes.byref(opt), ws.ptr, ws.nbytes, None))
        torch.cuda.synchronize()
        check_all(g, src, lambda q: (lv[q].cpu().numpy(), pa[q].cpu().numpy()), f"deep {variant}")
        counts.add(int(opt.levels))
    assert len(counts) == 1
