"""pm_exact_counts on both sides of every class bound of its kernels, against
closed forms: complete graphs (the lowest vertex has n - 1 forward neighbours:
64 | 256 | 1024), K_{2,q} (each hub's lower neighbours have degrees summing to
2 q: 384 | 3072 | 12288), and trees of q hubs of k leaves each, whose root
fills its table with q (k - 1) distinct ends and closes no cycle."""
from math import comb

import numpy as np
import pytest

from paper_1411_4942_amd import pathsamp as ps
from paper_1411_4942_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _exact(off, col):
    g = ps.Graph(torch.from_numpy(np.ascontiguousarray(off, np.int64)).cuda(),
                 torch.from_numpy(np.ascontiguousarray(col, np.int32)).cuda())
    return g.exact()


@pytest.mark.parametrize("n", [3, 4, 64, 65, 66, 257, 258])
def test_complete(n):
    print("[case] exact K", n, flush=True)
    e = _exact(*synth.complete(n))
    assert e["triangles"] == comb(n, 3)
    assert e["C"] == [0, 0, 0, 0, 0, 0, comb(n, 4)]
    assert e["N"][4] == 3 * comb(n, 4)


@pytest.mark.parametrize("q", [2, 3, 191, 192, 193, 1536, 1537, 6144, 6145])
def test_two_hubs(q):
    print("[case] exact K2,", q, flush=True)
    e = _exact(*synth.complete_bipartite(2, q))
    assert e["C"][4] == e["N"][4] == comb(q, 2)
    assert e["triangles"] == 0 and e["C"][5] == e["C"][6] == 0
    assert e["N"][1] == 2 * comb(q, 3)


@pytest.mark.parametrize("q,k", [(4, 95), (64, 6), (65, 5), (300, 10), (307, 10), (1228, 10), (1229, 10), (5, 3000)])
def test_tree_fills_tables(q, k):
    # root 0, hubs 1 .. q (degree k each), k - 1 leaves per hub
    hubs = np.arange(1, q + 1)
    leaves = q + 1 + np.arange(q * (k - 1))
    u = np.concatenate([np.zeros(q, np.int64), np.repeat(hubs, k - 1)])
    v = np.concatenate([hubs, leaves])
    print("[case] exact tree", q, k, flush=True)
    e = _exact(*synth.csr_from_edges(1 + q * k, u, v))
    assert e["C"][1] == comb(q, 3) + q * comb(k, 3)
    # 3-paths: over edges (root, hub) and (hub, leaf), (d_u - 1)(d_v - 1)
    assert e["C"][2] == q * (q - 1) * (k - 1)
    assert e["C"][3:] == [0, 0, 0, 0] and e["triangles"] == 0


# vertices above id 2^18 (the ids below are isolated) with more wedges than a
# table holds: counted with a bitmap, or range by range when too many repeat.
# 2^20 + 5000: the ids of a span's edge lie among the counted ones.
@pytest.mark.parametrize("n", [300000, (1 << 20) + 5000, 2200000])
@pytest.mark.parametrize("kind", ["few repeats", "hubs", "many repeats"])
def test_wedges_above_the_tables(n, kind):
    print("[case] exact bits", n, kind, flush=True)
    if kind == "hubs":  # K_{6,2500}
        off, col = synth.complete_bipartite(6, 2500)
        u, v = synth.edges_of(off, col)
        c4 = comb(6, 2) * comb(2500, 2)
    elif kind == "few repeats":  # a root over 200 hubs of 150 leaves, and 7 leaves shared by two hubs
        hubs = np.arange(1, 201)
        leaves = 201 + np.arange(200 * 150)
        u = np.concatenate([np.zeros(200, np.int64), np.repeat(hubs, 150), np.full(7, 2)])
        v = np.concatenate([hubs, leaves, leaves[:7]])
        c4 = comb(7, 2) + 7  # pairs of shared leaves, and a shared leaf with the root
    else:  # x over two sets of 4, each fully joined to 4000 others; x's own 4000 leaves put it on top
        a, b = np.arange(1, 9), 9 + np.arange(8000)
        leaves = 8009 + np.arange(4000)
        u = np.concatenate([np.zeros(8, np.int64), np.zeros(4000, np.int64), np.repeat(a[:4], 4000), np.repeat(a[4:], 4000)])
        v = np.concatenate([a, leaves, np.tile(b[:4000], 4), np.tile(b[4000:], 4)])
        c4 = 2 * comb(4, 2) * comb(4001, 2)
    e = _exact(*synth.csr_from_edges(n, u, v))
    assert e["N"][4] == c4
    assert e["triangles"] == 0
