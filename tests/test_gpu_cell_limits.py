"""LTM launches with more than four features at the limits of their work-groups:
a launch that is split because it passes 2^32 work-items, and pitches on both
sides of the 2^22 floats that 32-bit offsets take."""
import numpy as np
import pytest

from oracle import native
from paper_1308_1419_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_1308_1419_amd import tdmap  # noqa: E402


def test_second_launch():
    # rho 8, four block rows per work-group: 4 R (R + 1) / 2 work-groups of 64
    # threads with R = ceil(N / 32); the second launch does the columns from
    # 22008 on of the last 32 rows
    assert torch.cuda.is_available()
    N, d, rho = 185376, 5, 8
    R = -(-N // (4 * rho))
    first = ((1 << 32) - 1) // (rho * rho)
    assert first < 2 * R * (R + 1) < first + 4 * R
    X = synth.uniform_points(N, d, seed=31)
    size = N * (N + 1) // 2
    D = torch.empty(size + 64, dtype=torch.float32, device="cuda")
    top = N - 64  # the rows looked at; the others are the first launch's alone
    D[top * (top + 1) // 2:] = float("nan")
    tdmap.edm(torch.from_numpy(X).cuda(), layout="packed", rho=rho, out=D)
    torch.cuda.synchronize()
    rows = [top, N - 34, N - 33, N - 32, N - 31, N - 25, N - 24, N - 9, N - 8, N - 2, N - 1]
    tol = (d + 4) / 2 * 2.0 ** -23
    for i, ref in zip(rows, native.edm_rows(X, rows)):
        at = i * (i + 1) // 2
        got = D[at:at + i + 1].cpu().numpy()
        assert np.all(np.abs(got - ref) <= tol * ref), i
    assert not torch.isnan(D[top * (top + 1) // 2:size]).any()
    assert torch.isnan(D[size:]).all()
    del D
    torch.cuda.empty_cache()


@pytest.mark.parametrize("pitch", [(1 << 22) - 1, 1 << 22])
@pytest.mark.parametrize("rho", [8, 16, 32])
def test_pitches(rho, pitch):
    # 1460 points: past the size from which work-groups take four block rows
    assert torch.cuda.is_available()
    N, d = 1460, 7
    P = torch.from_numpy(synth.uniform_points(N, d, seed=rho)).cuda()
    lower = torch.tril(torch.ones((N, N), dtype=torch.bool, device="cuda"))
    ref = torch.full((N, N), float("nan"), device="cuda")
    tdmap.edm(P, strategy="utm", rho=rho, out=ref)
    buf = torch.empty(N * pitch, dtype=torch.float32, device="cuda").view(N, pitch)
    X = buf[:, :d]
    X.copy_(P)
    for layout in ("full", "packed"):  # points with the pitch
        got = tdmap.edm(X, layout=layout, rho=rho)
        assert torch.equal(got[lower] if layout == "full" else got, ref[lower]), layout
    buf[:, :N + 1] = float("nan")  # an output with the pitch
    tdmap.edm(P, rho=rho, out=buf, ldd=pitch)
    assert torch.equal(buf[:, :N].contiguous().view(torch.int32), ref.view(torch.int32))
    assert torch.isnan(buf[:, N]).all()
    del buf, X
    torch.cuda.empty_cache()
