"""Batches share the buffers of their draw-ordered runs: a second batch and
those after it take no more device memory than their own tables."""
import numpy as np
import pytest

from paper_1411_4942_amd import pathsamp as ps
from paper_1411_4942_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def test_batches_share_their_buffers():
    print("[case] batches share their buffers", flush=True)
    off, col = synth.erdos_renyi(1500, 9000, 21)
    g = ps.Graph(torch.from_numpy(np.ascontiguousarray(off, np.int64)).cuda(),
                 torch.from_numpy(np.ascontiguousarray(col, np.int32)).cuda())
    k = 1 << 21  # two samplers: a part of 2^22 samples, 0.1 GB
    want = g.count(k, k, seed=3)
    ps.release_cached_memory()
    torch.cuda.synchronize()
    batches, free = [], []
    for _ in range(6):
        b = ps.Batch([g], [ps.make_params(k, k, seed=3)], tune=(4096, 4))
        r = b.run()[0]
        assert r["tally_path"] == want["tally_path"] and r["tally_cent"] == want["tally_cent"]
        batches.append(b)
        torch.cuda.synchronize()
        free.append(torch.cuda.mem_get_info()[0])
    print("free MB:", [f >> 20 for f in free], flush=True)
    # a batch's own: the tile table (1024 tiles), the step's tables and the
    # tallies, each below one 2 MiB granule
    assert free[0] - free[-1] <= 5 * 5 * (2 << 20)
    for b in batches:
        b.destroy()
    g.destroy()


def _run(b, want):
    """One run, checked; was it draw-ordered?"""
    ps.profile_enable(True)
    r = b.run()[0]
    ordered = "sample_step" in ps.profile_read()
    ps.profile_enable(False)
    assert r["tally_path"] == want["tally_path"] and r["tally_cent"] == want["tally_cent"]
    return ordered


def test_memory_that_comes_back():
    """A run without memory for the order goes in id order; with memory again
    the runs are ordered again (after one failure one run is left out)."""
    print("[case] memory that comes back", flush=True)
    off, col = synth.erdos_renyi(1500, 9000, 21)
    g = ps.Graph(torch.from_numpy(np.ascontiguousarray(off, np.int64)).cuda(),
                 torch.from_numpy(np.ascontiguousarray(col, np.int32)).cuda())
    k = 1 << 23  # two samplers: a part of 2^24 samples, 0.3 GB
    want = g.count(k, k, seed=3)
    b = ps.Batch([g], [ps.make_params(k, k, seed=3)], tune=(4096, 4))
    assert _run(b, want)
    torch.cuda.empty_cache()
    ps.release_cached_memory()
    torch.cuda.synchronize()
    held = [torch.empty(torch.cuda.mem_get_info()[0] - (200 << 20), dtype=torch.uint8, device="cuda")]
    try:  # (more can be had than is reported free)
        for _ in range(64):
            held.append(torch.empty(256 << 20, dtype=torch.uint8, device="cuda"))
    except torch.cuda.OutOfMemoryError:
        pass
    print("held beyond the free memory: %d MB" % (256 * (len(held) - 1)), flush=True)
    assert not _run(b, want)
    del held
    torch.cuda.empty_cache()
    assert [_run(b, want) for _ in range(3)] == [False, True, True]
    b.destroy()
    g.destroy()
