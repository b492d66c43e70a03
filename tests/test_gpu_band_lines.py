"""Strips (rho = 256) on both sides of the lines of their rules (256 against
1024 or 512 columns, whole last tile row or not, fewer work-groups per CU) and
with last tile rows of every fill.  The 64-cell tiles use the same per-pair
function, so outputs are equal bit for bit, the cells that are not written
included (a NaN fill)."""
import pytest

from paper_1308_1419_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_1308_1419_amd import tdmap  # noqa: E402


def _buffer(N, layout):
    shape = (N, -(-N // 4) * 4) if layout == "full" else (N * (N - 1 if layout == "strict" else N + 1) // 2 + 8,)
    return torch.full(shape, float("nan"), dtype=torch.float32, device="cuda")


@pytest.mark.parametrize("d", [1, 3, 4])
@pytest.mark.parametrize("N", [2, 1026, 1537, 2049, 3071, 4578, 4579, 4580, 5633, 5792, 5793, 8688, 8689, 8690])
def test_lines_bitwise(N, d):
    assert torch.cuda.is_available()
    X = torch.from_numpy(synth.uniform_points(N, d, seed=3 * N + d)).cuda()
    for layout in ("full", "packed", "strict"):
        ref = tdmap.edm(X, layout=layout, rho=64, out=_buffer(N, layout))
        for strategy in ("ltm", "bb"):
            got = tdmap.edm(X, layout=layout, strategy=strategy, rho=256, out=_buffer(N, layout))
            assert torch.equal(got.view(torch.int32), ref.view(torch.int32)), (layout, strategy)
        parts = _buffer(N, layout)
        for shard in range(3):
            tdmap.edm_shard(X, shard, 3, layout=layout, rho=256, out=parts)
        assert torch.equal(parts.view(torch.int32), ref.view(torch.int32)), layout


@pytest.mark.parametrize("layout,d", [("full", 1), ("full", 3), ("packed", 3)])
def test_rows_past_the_last_point_cost_nothing(layout, d):
    # 4097 points begin a new tile row with their last one.  At the same pitch
    # they have the cells of 4096 and 0.05 % more; launching the whole tile row
    # took 1.20, 1.20 and 1.11 times as long, without it 0.99 to 1.00.  At most
    # 1.06.
    assert torch.cuda.is_available()
    sizes, ld = (4096, 4097), 4104
    X = {N: torch.from_numpy(synth.uniform_points(N, d, seed=N)).cuda() for N in sizes}
    out = torch.empty(4097 * ld, dtype=torch.float32, device="cuda")

    def burst(N):
        begin, end = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        begin.record()
        for _ in range(200):
            if layout == "full":
                tdmap.edm(X[N], rho=256, out=out.view(4097, ld), ldd=ld)
            else:
                tdmap.edm(X[N], layout=layout, rho=256, out=out)
        end.record()
        end.synchronize()
        return begin.elapsed_time(end)

    times = {N: [] for N in sizes}
    for _ in range(9):
        for N in sizes:
            times[N].append(burst(N))
    assert min(times[4097][1:]) <= 1.06 * min(times[4096][1:])
