"""Tallies at the edges of waves, blocks and launches, against the oracle:
the blocks' counts stored and summed by one kernel (pm_count in id order and
draw-ordered), the same launches with one atomic per block (pm_sample_async,
and more blocks than pm_count's scratch has rows for)."""
import numpy as np
import pytest

import oracle
from paper_1411_4942_amd import pathsamp as ps
from paper_1411_4942_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def pair():
    off, col = synth.erdos_renyi(400, 3000, 5)
    return ps.Graph(torch.from_numpy(off).cuda(), torch.from_numpy(col).cuda()), oracle.Graph(off, col)


@pytest.mark.parametrize("shape", [(1, 4), (4, 64), (2, 8), (1, 9)])  # 9: more rows than the scratch holds
@pytest.mark.parametrize("kp,kc", [(1, 1), (63, 65), (64, 64), (255, 257), (256, 1), (65537, 4095),
                                   (262145, 262143), (3, 0), (0, 700)])
def test_tallies_at_edges(pair, shape, kp, kc):
    g, og = pair
    want_p, want_c = og.sample_path(7, kp).tolist(), og.sample_centered(7, kc).tolist()
    print("[case] tally", shape, kp, kc, flush=True)
    ps.set_sampler_shape(*shape)
    try:
        r = g.count(kp, kc, seed=7)
        t = torch.full((16,), 77, dtype=torch.int64, device="cuda")
        g.sample_async(t, kp, kc, 7)
        t = t.cpu().tolist()
    finally:
        ps.set_sampler_shape(1, 4)
    assert (r["tally_path"], r["tally_cent"]) == (want_p, want_c)
    assert (t[:8], t[8:]) == (want_p, want_c)


@pytest.mark.parametrize("kp,kc", [(5000, 4097), (5000, 0), (5000, 100), (100, 5000)])
def test_tallies_draw_ordered(pair, kp, kc):
    g, og = pair
    want_p, want_c = og.sample_path(9, kp).tolist(), og.sample_centered(9, kc).tolist()
    print("[case] tally sorted", kp, kc, flush=True)
    ps.set_draw_order(True, 1000)
    try:
        r = g.count(kp, kc, seed=9)
    finally:
        ps.set_draw_order(True, 0)
    assert (r["tally_path"], r["tally_cent"]) == (want_p, want_c)
