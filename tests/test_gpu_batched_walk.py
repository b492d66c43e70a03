"""The batched sweep (rho = 1) where its walk changes step: sets just below and
above one chunk of 16384 positions, sets that fill the points' LDS exactly and
ones that exceed it, more empty sets in a row than the table holds, stretches
that end inside a set, an output that starts off a unit.  The 64-cell tiles
use the same per-pair function, so the outputs are equal bit for bit."""
import numpy as np
import pytest

from paper_1308_1419_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_1308_1419_amd import tdmap  # noqa: E402

SIZES = {
    "chunk": [180, 181, 182, 0, 1, 255, 256, 257, 180, 2, 181],
    "empty": [3] + [0] * 2500 + [200, 0, 0, 5] + [0] * 1023 + [190] + [0] * 1024 + [7],
    "tiny": [1, 2, 0, 3] * 9000,
    "growing": list(range(0, 700, 3)),
    "large": [4096, 3, 4096, 5462, 20, 5461, 2731, 2730, 16385, 64, 8193, 1],
}


@pytest.mark.parametrize("shift", [0, 5])
@pytest.mark.parametrize("d", [1, 2, 3, 4])
@pytest.mark.parametrize("which", list(SIZES))
def test_walk_bitwise(which, d, shift):
    assert torch.cuda.is_available()
    n = np.asarray(SIZES[which], dtype=np.int64)
    po = np.concatenate([[0], np.cumsum(n)]).astype(np.int64)
    oo = (shift + np.concatenate([[0], np.cumsum(n * (n + 1) // 2)])).astype(np.int64)
    X = torch.from_numpy(synth.uniform_points(int(po[-1]), d, seed=d)).cuda()
    pod, ood = torch.from_numpy(po).cuda(), torch.from_numpy(oo).cuda()
    outs = []
    for rho in (64, 1):
        out = torch.full((int(oo[-1]) + 64,), float("nan"), dtype=torch.float32, device="cuda")
        tdmap.edm_batched(X, pod, ood, rho=rho, out=out)
        outs.append(out.view(torch.int32))
    torch.cuda.synchronize()
    assert torch.equal(outs[0], outs[1])
    assert bool(torch.isnan(outs[1].view(torch.float32)[:shift]).all())
