"""The stable radix sort and the ingest's half-sorts at the edges of tiles,
histogram chunks and digit widths, seen through what they build: the CSR of
an edge list and the prepared graph's relabelled arrays, against the oracle."""
import numpy as np
import pytest

import oracle
from oracle import ingest as oracle_ingest
from paper_1411_4942_amd import pathsamp as ps
from paper_1411_4942_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _pairs(n, pairs, seed):
    rng = np.random.Generator(np.random.PCG64(seed))
    # skewed ends (squares crowd the low ids), loops and repeats among them
    u = (n * rng.random(pairs) ** 2).astype(np.int32)
    v = (n * rng.random(pairs) ** 2).astype(np.int32)
    return u, v


# one tile is 8192 pairs; digits are 1 pass up to 11 bits, 2 up to 22, 3 above
@pytest.mark.parametrize("n,pairs", [(1, 5), (2, 9), (256, 8191), (257, 8192), (2048, 8193), (2049, 16384),
                                     (70000, 65537), (1 << 22, 30000), ((1 << 22) + 1, 30000), (30000000, 20000),
                                     (100000, 9000001)])
def test_ingest_edges(n, pairs):
    u, v = _pairs(n, pairs, n + pairs)
    print("[case] ingest", n, pairs, flush=True)
    off, col = ps.csr_from_edges(n, torch.from_numpy(u).cuda(), torch.from_numpy(v).cuda())
    lo, hi = np.minimum(u, v).astype(np.int64), np.maximum(u, v).astype(np.int64)
    key = np.unique(lo[lo != hi] * n + hi[lo != hi])
    if pairs < 100000 and n < 100000:
        want_off, want_col = oracle_ingest.csr_from_edges(n, u, v)
        assert np.array_equal(off.cpu().numpy(), want_off) and np.array_equal(col.cpu().numpy(), want_col)
    both = np.sort(np.concatenate([key, key % n * n + key // n]))
    assert np.array_equal(col.cpu().numpy(), both % n)
    assert np.array_equal(off.cpu().numpy(), np.searchsorted(both, np.arange(n + 1, dtype=np.int64) * n))


@pytest.mark.parametrize("n,m", [(2, 1), (1025, 4096), (2049, 4097), (5000, 300000), (9000, 45000)])
def test_prepared_arrays_at_sort_edges(n, m):
    off, col = synth.erdos_renyi(n, m, n)
    print("[case] prep", n, m, flush=True)
    g = ps.Graph(torch.from_numpy(off).cuda(), torch.from_numpy(col).cuda())
    og, x = oracle.Graph(off, col), g.export()
    assert np.array_equal(x["off"], og.off) and np.array_equal(x["col"], og.col) and np.array_equal(x["rank"], og.rank)
    assert np.array_equal(x["p_tau"], og.p_tau) and np.array_equal(x["p_lam"], og.p_lam)
