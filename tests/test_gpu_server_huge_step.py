"""A server step beyond what its tile table holds is refused, in draw order as
in id order: pilots of 2^50 samples and more, also where the samples of the
step's requests sum to 2^64."""
import numpy as np
import pytest

from paper_1411_4942_amd import pathsamp as ps
from paper_1411_4942_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("order", [True, False])
@pytest.mark.parametrize("k_pilot", [1 << 50, 1 << 62, 1 << 63])
def test_step_too_large(k_pilot, order):
    print("[case] huge step", k_pilot, order, flush=True)
    off, col = synth.erdos_renyi(1500, 9000, 21)
    o, c = (torch.from_numpy(np.ascontiguousarray(off, np.int64)).cuda(),
            torch.from_numpy(np.ascontiguousarray(col, np.int32)).cuda())
    ps.set_draw_order(order, 0)
    srv = ps.Server(k_pilot=k_pilot, k_max=k_pilot)
    try:
        g = srv.add_graph(o, c)
        with pytest.raises(ps.PathSampError, match="step too large") as e:
            srv.wait(srv.submit(g, rel_err=0.1, seed=1), timeout_ms=60000)
        assert e.value.status == ps.PM_EINVAL
        r, _ = srv.wait(srv.submit(g, k_path=5000, k_cent=4000, seed=2), timeout_ms=60000)  # and the server goes on
        want = ps.Graph(o, c).count(5000, 4000, seed=2)
        assert r["tally_path"] == want["tally_path"] and r["tally_cent"] == want["tally_cent"]
    finally:
        srv.destroy()
        ps.set_draw_order(True, 0)
