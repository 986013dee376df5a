"""Draw-ordered runs of a batch: every graph's tallies equal its own count,
for budgets on both sides of the order's threshold and changed between runs.
Integer tallies: compared exactly."""
import numpy as np
import pytest

from paper_1411_4942_amd import pathsamp as ps
from paper_1411_4942_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def graphs():
    csr = [synth.erdos_renyi(1500, 9000, 21), synth.star(9), synth.cycle(12), synth.complete(5),
           synth.chung_lu(4000, 30000, 2.3, 300.0, 22)]
    return [ps.Graph(torch.from_numpy(np.ascontiguousarray(o, np.int64)).cuda(),
                     torch.from_numpy(np.ascontiguousarray(c, np.int32)).cuda()) for o, c in csr]


@pytest.fixture(autouse=True)
def default_order():
    yield
    ps.set_draw_order(True, 0)


def check(graphs, b, params):
    got = b.run()
    for g, p, r in zip(graphs, params, got):
        want = g.count(p.k_path, p.k_cent, seed=p.seed)
        assert r["tally_path"] == want["tally_path"] and r["tally_cent"] == want["tally_cent"]
        assert r["est"] == want["est"] and r["lo"] == want["lo"] and r["hi"] == want["hi"]


@pytest.mark.parametrize("tune", [None, (1024, 1), (4096, 8)])
def test_runs_equal_their_own_counts(graphs, tune):
    big = [ps.make_params(5000 + 77 * i, 4000 + 33 * i, seed=i) for i in range(len(graphs))]
    small = [ps.make_params(1 + i, 64 if i % 2 else 0, seed=9 + i) for i in range(len(graphs))]
    b = ps.Batch(graphs, big, tune=tune)
    for order_min in (1, 30000, 1 << 30):  # ordered; ordered for the large budgets alone; id order
        ps.set_draw_order(True, order_min)
        for params in (big, small, big):
            b.set_params(params)
            check(graphs, b, params)
    b.destroy()


def test_many_graphs(graphs):
    """More (graph, sampler) pairs than one part counts."""
    n = 300
    gs = [graphs[(0, 4)[i % 2]] for i in range(n)]
    params = [ps.make_params(100 + i, 90 + i, seed=i) for i in range(n)]
    ps.set_draw_order(True, 1)
    b = ps.Batch(gs, params, tune=(1024, 4))
    check(gs, b, params)
    b.destroy()
