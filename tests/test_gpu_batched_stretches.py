"""The batched sweep (rho = 1) with enough positions that every work-group owns
well over a chunk (16384 positions) of the walk: full and quarter chunks of sets
just below and above one chunk, the change of the staged points from set to
set, and tables that fill up with sets.  The 64-cell tiles use the same per-pair
function, so the outputs are equal bit for bit."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_1308_1419_amd import tdmap  # noqa: E402

UNIT, CHUNK = 1024, 16384
# a set of 180 points has 16290 cells, of 181 points 16471
SIZES = {
    "chunk": [180, 181, 182, 0, 1, 255, 256, 257, 180, 2, 181] * 300,
    "chunk_and_tiny": [181, 1, 3, 0, 2, 400] * 900,
    "tiny": [1, 2, 0, 3, 5] * 200000,
    "pairs": [2] * 1500000,
    "full_table": ([4] * 1023 + [181] + [4] * 1024 + [182]) * 500,
}


@pytest.mark.parametrize("shift", [0, 3])
@pytest.mark.parametrize("d", [1, 2, 3, 4])
@pytest.mark.parametrize("which", list(SIZES))
def test_stretches_bitwise(which, d, shift):
    assert torch.cuda.is_available()
    n = np.asarray(SIZES[which], dtype=np.int64)
    po = np.concatenate([[0], np.cumsum(n)]).astype(np.int64)
    oo = (shift + np.concatenate([[0], np.cumsum(n * (n + 1) // 2)])).astype(np.int64)
    groups = 2 * torch.cuda.get_device_properties(0).multi_processor_count
    stretch = (int(oo[-1]) - shift) // groups
    assert stretch > (2 * CHUNK if "chunk" in which or which == "full_table" else 4 * UNIT)
    X = torch.rand((int(po[-1]), d), device="cuda", generator=torch.Generator("cuda").manual_seed(d))
    pod, ood = torch.from_numpy(po).cuda(), torch.from_numpy(oo).cuda()
    outs = []
    for rho in (64, 1):
        out = torch.full((int(oo[-1]) + 64,), float("nan"), dtype=torch.float32, device="cuda")
        tdmap.edm_batched(X, pod, ood, rho=rho, out=out)
        outs.append(out.view(torch.int32))
    torch.cuda.synchronize()
    assert torch.equal(outs[0], outs[1])
    bits = outs[1].view(torch.float32)
    assert bool(torch.isnan(bits[:shift]).all()) and bool(torch.isnan(bits[int(oo[-1]):]).all())
    assert not bool(torch.isnan(bits[shift:int(oo[-1])]).any())
