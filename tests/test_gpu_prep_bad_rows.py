"""Preparation refuses a hub row of equal columns as fast as it builds a sound
one: no row hash is built of rows that fail a check (equal keys would each
probe past all the others).

Bound: after the check the row hash's kernels read one word and end, so their
time is at most the sound graph's; half a millisecond is left for the timer
and a first launch.  6000 equal keys probed one after the other are 1.8e7
LDS operations of one block, all lanes on one address: 7 ms."""
import numpy as np
import pytest

from paper_1411_4942_amd import pathsamp as ps
from paper_1411_4942_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _timed(off, col):
    """The build's result (None: refused) and its row hash's milliseconds."""
    ps.profile_enable(True)
    try:
        g, err = ps.Graph(off, col), None
    except ps.PathSampError as e:
        g, err = None, e
    ms = {k: v[1] for k, v in ps.profile_read().items()}["rowhash"]
    ps.profile_enable(False)
    return g, err, ms


# degrees of the hash's classes: many rows a block, one window, several, the
# hub rows of the row build
@pytest.mark.parametrize("d", [1000, 3000, 6000, 20000, 100000])
@pytest.mark.parametrize("fault,match", [("range", "column is not a vertex id"), ("order", "not strictly ascending"),
                                         ("loop", "self-loop")])
def test_hub_of_equal_columns(d, fault, match):
    print("[case] bad hub row", d, fault, flush=True)
    off, col = synth.star(d)
    n, hub = len(off) - 1, int(np.argmax(np.diff(off)))
    assert off[hub + 1] - off[hub] >= d - 1
    t_off = torch.from_numpy(np.ascontiguousarray(off, np.int64)).cuda()
    good, err, good_ms = _timed(t_off, torch.from_numpy(np.ascontiguousarray(col, np.int32)).cuda())
    assert err is None
    good.destroy()
    bad = np.array(col, np.int32)
    bad[off[hub]:off[hub + 1]] = {"range": n, "order": (hub + 1) % n, "loop": hub}[fault]
    g, err, ms = _timed(t_off, torch.from_numpy(bad).cuda())
    assert g is None and err.status == ps.PM_EGRAPH
    assert match in str(err)
    print("row hash of the sound graph %.3f ms, of the refused one %.3f ms" % (good_ms, ms), flush=True)
    assert ms <= good_ms + 0.5
