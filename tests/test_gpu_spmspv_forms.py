"""The masked product where its work is split differently: vectors of one entry to
more columns than waves, columns on both sides of the chunk length, duplicate
and empty columns, an empty vector, a bad vector followed by a good one on the
same workspace, and a graph of so many vertices that the output offsets take a
pass of their own."""
import numpy as np
import pytest

import graphgen
from gpu_common import need_gpu, say

pytestmark = pytest.mark.gpu


def _reference(ptr, idx, n, x, v, semiring, visited):
    deg = ptr[x + 1] - ptr[x]
    rows = np.concatenate([idx[ptr[j]:ptr[j + 1]] for j in x]) if len(x) else np.zeros(0, int)
    val = np.repeat(v, deg)
    keep = ~visited[rows]
    rows, val = rows[keep], val[keep]
    y = np.unique(rows)
    out = np.full(n, np.iinfo(np.int64).max) if semiring.startswith("min") else np.zeros(n, np.int64)
    if semiring == "arithmetic":
        np.add.at(out, rows, val)
    elif semiring == "boolean":
        np.maximum.at(out, rows, (val != 0).astype(np.int64))
    else:
        np.minimum.at(out, rows, val + (semiring == "min_plus"))
    return y, out[y]


@pytest.mark.parametrize("semiring", ["boolean", "arithmetic", "min_plus", "min_select"])
@pytest.mark.parametrize("nx", [0, 1, 63, 4097, 30000])
def test_product_forms(semiring, nx):
    import torch
    P = need_gpu()
    rng = np.random.default_rng(nx)
    n = 9001
    deg = np.concatenate([rng.integers(0, 30, n - 6), [511, 512, 513, 1024, 1025, 8000]])
    g = graphgen.from_edges(n, np.repeat(np.arange(n), deg), rng.integers(0, n, deg.sum()), directed=True)
    G = P.Graph.from_graphgen(g)
    x = rng.integers(0, n, nx).astype(np.int32)
    x[:min(6, nx)] = np.arange(n - 6, n)[:min(6, nx)]
    v = rng.integers(0, 1 << 40, nx)
    visited = rng.random(n) < 0.4
    words = np.packbits(np.concatenate([visited, np.zeros(-n % 32, bool)]), bitorder="little").view(np.int32)
    ws = P.Workspace(P.spmspv_workspace_size(G, max(nx, 1)))
    ws.buf.zero_()
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    want_i, want_v = _reference(g.ptr.astype(np.int64), g.idx, n, x.astype(np.int64), v, semiring, visited)
    for bad in (False, True, False):
        say(f"[product] {semiring} nx={nx} bad={bad}")
        xi = x.copy()
        if bad:
            if nx == 0:
                continue
            xi[nx // 2] = n
            with pytest.raises(P.BfsError):
                P.masked_spmspv(G, semiring, dev(xi), dev(v), row_mask=dev(words), row_complement=True, workspace=ws)
            continue
        yi, yv = P.masked_spmspv(G, semiring, dev(xi), dev(v), row_mask=dev(words), row_complement=True, workspace=ws)
        assert np.array_equal(yi.cpu().numpy(), want_i) and np.array_equal(yv.cpu().numpy(), want_v)


def test_product_many_output_blocks():
    import torch
    P = need_gpu()
    n = 4097 * 8192 + 5                        # 4,098 blocks of the output passes
    ptr = np.minimum(np.arange(n + 1, dtype=np.int32), n - 1)           # a directed path
    G = P.Graph.from_csr(n, ptr, np.arange(1, n, dtype=np.int32), np.maximum(np.arange(n + 1, dtype=np.int32) - 1, 0),
                         np.arange(n - 1, dtype=np.int32), directed=True)
    x = np.unique(np.concatenate([np.array([0, n - 2]), np.random.default_rng(1).integers(0, n - 1, 1000)])).astype(np.int32)
    say("[product] many output blocks")
    yi, yv = P.masked_spmspv(G, "min_select", torch.from_numpy(x).cuda(), torch.from_numpy(x.astype(np.int64)).cuda())
    assert np.array_equal(yi.cpu().numpy(), x + 1) and np.array_equal(yv.cpu().numpy(), x)
