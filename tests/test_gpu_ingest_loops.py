"""Edge lists that leave no pair: loops alone, at sizes whose buffers are
allocations of their own, and one vertex.  Compared exactly."""
import numpy as np
import pytest

from oracle import ingest
from paper_1411_4942_amd import pathsamp as ps

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n,e", [(1, 1), (1, 1 << 20), (2, 1025), (1 << 20, 1 << 20), (3000, (1 << 20) + 1)])
def test_loops_leave_empty_rows(n, e):
    print("[case] ingest loops", n, e, flush=True)
    v = (np.arange(e, dtype=np.int64) * 7919 % n).astype(np.int32)
    want_off, want_col = ingest.csr_from_edges(n, v, v)
    off, col = ps.csr_from_edges(n, torch.from_numpy(v).cuda(), torch.from_numpy(v).cuda())
    assert np.array_equal(off.cpu().numpy(), want_off) and col.numel() == len(want_col) == 0
    g = ps.Graph.from_edges(n, torch.from_numpy(v).cuda(), torch.from_numpy(v).cuda())
    assert g.info()["n"] == n and g.info()["m"] == 0
    g.destroy()
