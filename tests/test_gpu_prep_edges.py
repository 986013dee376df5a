"""Preparation on both sides of its one-block scans (offsets: up to 32768
vertices; segments of 1024 slots: 4096 per round) and with isolated vertices,
against the oracle's arrays and totals; an input with several faults reports
the row's own fault and not the asymmetry it causes."""
import numpy as np
import pytest

import oracle
from paper_1411_4942_amd import pathsamp as ps
from paper_1411_4942_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _dev(off, col):
    return (torch.from_numpy(np.ascontiguousarray(off, np.int64)).cuda(),
            torch.from_numpy(np.ascontiguousarray(col, np.int32)).cuda())


@pytest.mark.parametrize("n,m", [(1, 0), (3, 2), (4095, 9000), (8192, 9000), (8193, 9000), (32767, 50000),
                                 (32768, 50000), (32769, 50000), (40000, 2097152 + 600)])
def test_scans_at_their_edges(n, m):
    print("[case] prep edges", n, m, flush=True)
    if m:
        off, col = synth.erdos_renyi(n, m, n)
    else:
        off, col = synth.empty(n)
    g, og = ps.Graph(*_dev(off, col)), oracle.Graph(off, col)
    x, info = g.export(), g.info()
    for f in ("off", "col", "rank", "p_tau", "p_lam"):
        assert np.array_equal(x[f], getattr(og, f)), f
    deg = np.diff(off)
    assert info["isolated"] == int((deg == 0).sum()) and info["dmax"] == int(deg.max())
    assert (info["W"], info["Lambda"], info["N1"]) == (og.W, og.Lam, og.N1)


def test_row_faults_before_the_asymmetry():
    off, col = synth.erdos_renyi(500, 3000, 1)
    bad = col.copy()
    v = int(np.argmax(np.diff(off)))
    bad[off[v]] = 500  # not a vertex id; its row no longer matches the others either
    with pytest.raises(ps.PathSampError, match="column is not a vertex id") as e:
        ps.Graph(*_dev(off, bad))
    assert e.value.status == ps.PM_EGRAPH
    bad = col.copy()
    bad[off[v]:off[v] + 2] = bad[off[v]:off[v] + 2][::-1]
    with pytest.raises(ps.PathSampError, match="not strictly ascending"):
        ps.Graph(*_dev(off, bad))
    g = ps.Graph(*_dev(off, col))  # and a sound graph builds after them
    assert g.info()["m"] == 3000
