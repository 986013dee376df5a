"""A slot's row in the weights pass: from its segment's first row (segments of
1024 slots) and the rows that start inside it.  Segments full of one-slot
rows, rows over many segments, row starts on and beside segment boundaries, a
last segment of one slot; the prefixes and the records (through the samplers)
against the oracle, exactly."""
import numpy as np
import pytest

import oracle
from paper_1411_4942_amd import pathsamp as ps

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _csr(n, edges):
    e = np.array(edges, dtype=np.int64).reshape(-1, 2)
    both = np.concatenate([e, e[:, ::-1]])
    both = both[np.lexsort((both[:, 1], both[:, 0]))]
    return np.searchsorted(both[:, 0], np.arange(n + 1)).astype(np.int64), both[:, 1].astype(np.int32)


def _pairs(k):  # 2k one-slot rows, and a path so that something is sampled
    e = [(2 * i, 2 * i + 1) for i in range(k)]
    return 2 * k + 5, e + [(2 * k + i, 2 * k + i + 1) for i in range(4)]


def _hubs(leaves, hubs):  # one-slot and hubs-slot rows, then rows of `leaves` slots
    return leaves + hubs + 1, ([(i, leaves + h) for i in range(leaves) for h in range(hubs)] +
                               [(leaves + h, leaves + hubs) for h in range(hubs)])


def _cycles(k, length):
    return k * length, [(c * length + i, c * length + (i + 1) % length) for c in range(k) for i in range(length)]


CASES = {"one-slot rows": _pairs(2050), "row starts at 1024": _cycles(256, 4), "one slot less": _pairs(508),
         "1025 slots": _hubs(511, 1), "a hub": _hubs(5000, 1), "three hubs": _hubs(1024, 3), "cycles": _cycles(700, 5)}


@pytest.mark.parametrize("name", list(CASES))
def test_rows_of_slots(name):
    print("[case]", name, flush=True)
    off, col = _csr(*CASES[name])
    g = ps.Graph(torch.from_numpy(off).cuda(), torch.from_numpy(col).cuda())
    og, x = oracle.Graph(off, col), g.export()
    for f in ("off", "col", "p_tau", "p_lam"):
        assert np.array_equal(x[f], getattr(og, f)), f
    assert (g.info()["W"], g.info()["Lambda"]) == (og.W, og.Lam)
    k = 5000
    res = g.count(k, k, seed=7)
    assert res["tally_path"] == (og.sample_path(7, k).tolist() if og.R_tau else [0] * 8)
    assert res["tally_cent"] == (og.sample_centered(7, k).tolist() if og.R_lam else [0] * 8)
