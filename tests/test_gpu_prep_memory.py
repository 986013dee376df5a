"""A graph that fails a row check is refused for that also where there is no
memory for the rest of its build: the device's memory is held up to what the
rows need (the row hash behind them is one allocation of 4.2 GB, of which some
2 GB are left), and the build of a sound graph then runs out of memory."""
import pytest

from paper_1411_4942_amd import pathsamp as ps

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

N, HALF = 1 << 16, 4000  # the circulant graph v ~ v +- 1 .. HALF: 5.2e8 slots


def _circulant():
    step = torch.arange(1, HALF + 1, device="cuda", dtype=torch.int32)
    step = torch.cat([step, N - step])
    cols = torch.empty((N, 2 * HALF), dtype=torch.int32, device="cuda")
    for v in range(0, N, 1024):
        rows = torch.arange(v, v + 1024, device="cuda", dtype=torch.int32)
        cols[v:v + 1024] = ((rows[:, None] + step[None, :]) % N).sort(dim=1).values
    return torch.arange(N + 1, device="cuda", dtype=torch.int64) * (2 * HALF), cols.view(-1)


def test_bad_rows_before_no_memory():
    print("[case] bad rows without memory", flush=True)
    off, cols = _circulant()
    slots = cols.numel()
    torch.cuda.empty_cache()
    ps.release_cached_memory()
    # until the row hash: columns 4, records 16, the ladder, the sort's scratch
    # and the vertices' arrays: 20.7 bytes a slot
    need = int(20.7 * slots)
    free, _ = torch.cuda.mem_get_info()
    held = torch.empty(free - need - (2 << 30), dtype=torch.uint8, device="cuda")
    try:
        with pytest.raises(ps.PathSampError) as e:
            ps.Graph(off, cols)
        assert e.value.status == ps.PM_ENOMEM
        cols[5 * 2 * HALF + 7] = cols[5 * 2 * HALF + 6]  # an edge twice
        with pytest.raises(ps.PathSampError, match="not strictly ascending") as e:
            ps.Graph(off, cols)
        assert e.value.status == ps.PM_EGRAPH
    finally:
        del held
        torch.cuda.empty_cache()
        ps.release_cached_memory()
    torch.cuda.synchronize()
