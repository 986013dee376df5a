"""Draw-ordered server steps: the results of requests that share steps equal
those of the id order and of each request run alone, whatever the graphs,
budgets, parts and chunks.  Integer tallies: compared exactly."""
import numpy as np
import pytest

from paper_1411_4942_amd import pathsamp as ps
from paper_1411_4942_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

GRAPHS = [
    synth.erdos_renyi(1500, 9000, 21),
    synth.star(9),  # no sampler draws
    synth.cycle(12),  # only the 3-path sampler
    synth.complete(5),  # weights of a few units: many draws share a rank
    synth.chung_lu(4000, 30000, 2.3, 300.0, 22),
    synth.rmat(11, 16, seed=23),
]


@pytest.fixture(scope="module")
def dev():
    return [(torch.from_numpy(np.ascontiguousarray(o, np.int64)).cuda(),
             torch.from_numpy(np.ascontiguousarray(c, np.int32)).cuda()) for o, c in GRAPHS]


@pytest.fixture(autouse=True)
def default_order():
    yield
    ps.set_draw_order(True, 0)


def run(dev, reqs, **cfg):
    srv = ps.Server(**cfg)
    ids = [srv.add_graph(o, c) for o, c in dev]
    tickets = [srv.submit(ids[g], k_path=kp, k_cent=kc, seed=seed) for g, kp, kc, seed in reqs]
    out = [srv.wait(t)[0] for t in tickets]
    srv.destroy()
    return [(r["tally_path"], r["tally_cent"]) for r in out]


def check(dev, reqs, **cfg):
    ps.set_draw_order(True, 1)
    got = run(dev, reqs, **cfg)
    ps.set_draw_order(False)
    solo = [ps.Graph(o, c) for o, c in dev]
    for (g, kp, kc, seed), (tp, tc) in zip(reqs, got):
        want = solo[g].count(kp, kc, seed=seed)
        assert tp == want["tally_path"] and tc == want["tally_cent"], (g, kp, kc, seed)


# one sample; one wave and one more; a sampler without work; several requests on a graph, one seed twice
@pytest.mark.parametrize("reqs", [
    [(0, 1, 0, 1)],
    [(0, 64, 65, 1)],
    [(0, 0, 257, 1), (4, 1000, 0, 2)],
    [(g, 1 + 977 * i % 3001, 1 + 641 * i % 2503, i // 2) for i, g in enumerate([5, 0, 3, 2, 4, 0, 5, 5, 1, 3, 4, 0])],
], ids=["one", "wave", "one-sided", "mixed"])
def test_requests_equal_their_own_counts(dev, reqs):
    check(dev, reqs)


def test_many_requests(dev):
    """As many chunks as a part counts, and more."""
    for n in (256, 300):
        check(dev, [(i % len(GRAPHS), 100 + i, 90 + i, i) for i in range(n)], max_active=n)


@pytest.mark.parametrize("k", [(1 << 24) - 1, (1 << 24) + 4096])
def test_parts(dev, k):
    """A request cut by the parts of a step, beside smaller ones."""
    check(dev, [(0, 5000, 300, 3), (4, k, 70000, 4), (5, 100, 100, 5)], step_samples=1 << 26)


def test_pilot_and_sized_budgets(dev):
    out = []
    for on in (True, False):
        ps.set_draw_order(on, 1)
        srv = ps.Server(k_pilot=20000)
        ids = [srv.add_graph(o, c) for o, c in dev]
        t = [srv.submit(ids[g], rel_err=0.1, seed=s) for s, g in enumerate([0, 4, 5, 4, 0])]
        out.append([srv.wait(x) for x in t])
        srv.destroy()
    for (a, sa), (b, sb) in zip(*out):
        assert a["tally_path"] == b["tally_path"] and a["tally_cent"] == b["tally_cent"]
        assert (sa["k_path"], sa["k_cent"]) == (sb["k_path"], sb["k_cent"])
