"""LTM launches with more than four features and at least 2^20 cells: a
work-group does several block rows of one block column.  Every cell has the
bits that UTM's pair-by-pair launch gives, and nothing else is written; the
sizes lie at the lines of the rule and around whole groups of block rows."""
import numpy as np
import pytest

from paper_1308_1419_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_1308_1419_amd import tdmap  # noqa: E402


@pytest.mark.parametrize("rho", [8, 16, 32])
@pytest.mark.parametrize("N,d", [(1448, 17), (1449, 16), (1472, 5), (1537, 33), (2047, 20), (2048, 8),
                                 (3547, 7), (3548, 16), (3584, 31), (3841, 12)])
def test_rows_bitwise(N, d, rho):
    assert torch.cuda.is_available()
    X = synth.uniform_points(N, d + 3, seed=7 * d + N)
    Xd = torch.from_numpy(X).cuda()[:, 1:d + 1]  # ldx = d + 3, 4 bytes past the base
    ld = N + 3
    lower = torch.tril(torch.ones((N, N), dtype=torch.bool, device="cuda"))
    for layout in ("full", "packed"):
        outs = []
        for s in ("utm", "ltm"):
            size = N * ld if layout == "full" else N * (N + 1) // 2
            D = torch.full((size + 64,), float("nan"), dtype=torch.float32, device="cuda")
            out = D[:size].view(N, ld) if layout == "full" else D[:size]
            tdmap.edm(Xd, layout=layout, strategy=s, rho=rho, out=out)
            torch.cuda.synchronize()
            outs.append(D)
        assert torch.equal(outs[0].view(torch.int32), outs[1].view(torch.int32)), layout
        assert torch.isnan(outs[1][size:]).all(), layout
        got = outs[1][:size].view(N, ld)[:, :N][lower] if layout == "full" else outs[1][:size]
        assert not torch.isnan(got).any(), layout
    # the last layout is packed: its first and last rows against FP64
    tol = (d + 4) / 2 * 2.0 ** -23
    P = np.ascontiguousarray(X[:, 1:d + 1])
    for i in (0, 1, 255, N // 2, N - 1):
        ref = np.sqrt(((P[i].astype(np.float64) - P[:i + 1].astype(np.float64)) ** 2).sum(1))
        row = got[i * (i + 1) // 2:(i + 1) * (i + 2) // 2].cpu().numpy()
        assert np.all(np.abs(row - ref) <= tol * ref), i
