"""Strips (rho = 256) at the edges of their shapes: tiles of 256, 512 and 1024
columns, strips of 2 to 8 rows, the last row and column of each, outputs that
allow 16-byte stores and outputs that do not, points with and without a pitch,
and a size past the one where fewer work-groups share a CU.  The 64-cell
tiles take the same per-pair function on another split, so the outputs are
equal bit for bit, the cells outside the triangle included (a NaN fill)."""
import numpy as np
import pytest

from paper_1308_1419_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_1308_1419_amd import tdmap  # noqa: E402


def _run(X, layout, strategy, rho, ld, shift):
    N = X.shape[0]
    size = N * ld if layout == "full" else N * (N + 1) // 2
    buf = torch.full((size + 8,), float("nan"), dtype=torch.float32, device="cuda")
    out = buf[shift:shift + size]
    tdmap.edm(X, layout=layout, strategy=strategy, rho=rho,
              out=out.view(N, ld) if layout == "full" else out, ldd=ld if layout == "full" else None)
    torch.cuda.synchronize()
    return buf.view(torch.int32)


@pytest.mark.parametrize("d", [1, 2, 3, 4])
@pytest.mark.parametrize("N", [1, 3, 255, 257, 511, 512, 513, 1023, 1025, 1030, 2047, 2050, 6001])
def test_strips_bitwise(N, d):
    assert torch.cuda.is_available()
    P = torch.from_numpy(synth.uniform_points(N, d + 2, seed=5 * N + d)).cuda()
    for X in (P[:, :d].contiguous(), P[:, 1:d + 1]):
        for layout, ld, shift in (("full", -(-N // 4) * 4, 0), ("full", -(-N // 4) * 4, 1),
                                  ("full", N + 1 - N % 2, 0), ("packed", 0, 0), ("packed", 0, 3),
                                  ("strict", 0, 0)):
            ref = _run(X, layout, "ltm", 64, ld, shift)
            for strategy in ("ltm", "bb"):
                got = _run(X, layout, strategy, 256, ld, shift)
                assert torch.equal(got, ref), (layout, ld, shift, strategy)
