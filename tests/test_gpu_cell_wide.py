"""One-cell-per-thread launches with more than four features: LTM, BB and REC
stage their points per block; UTM reads them in place, pair by pair.  All add
the squared differences in feature order, so they agree bit for bit, and the
values meet the FP64 oracle within (d + 4) / 2 units of FP32 roundoff (d + 1
roundings of non-negative terms under the root, one in each difference)."""
import numpy as np
import pytest

from oracle import edm as oedm
from paper_1308_1419_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_1308_1419_amd import tdmap  # noqa: E402


@pytest.mark.parametrize("rho", [8, 16, 32])
@pytest.mark.parametrize("N,d", [(1, 5), (2, 16), (31, 17), (32, 15), (33, 32), (64, 33), (97, 5),
                                 (257, 20), (300, 47), (129, 130)])
def test_wide_cells_bitwise(N, d, rho):
    assert torch.cuda.is_available()
    X = synth.uniform_points(N, d + 3, seed=11 * d + N)
    Xd = torch.from_numpy(X).cuda()[:, 2:d + 2]  # ldx = d + 3, 8 bytes past the base
    ref = oedm.edm64_full(np.ascontiguousarray(X[:, 2:d + 2]))
    lower = np.tril(np.ones((N, N), dtype=bool))
    ld = N + 5
    first = {}
    for layout in ("full", "packed"):
        for s in ("utm", "ltm", "bb", "rec"):
            size = N * ld if layout == "full" else N * (N + 1) // 2
            D = torch.full((size + 64,), float("nan"), dtype=torch.float32, device="cuda")
            out = D[:size].view(N, ld) if layout == "full" else D[:size]
            tdmap.edm(Xd, layout=layout, strategy=s, rho=rho, out=out)
            torch.cuda.synchronize()
            h = D.cpu().numpy()
            assert np.isnan(h[size:]).all(), (layout, s)
            bits = first.setdefault(layout, h.view(np.int32))
            assert np.array_equal(h.view(np.int32), bits), (layout, s)
        got = h[:size].reshape(N, ld)[:, :N][lower] if layout == "full" else h[:size]
        tol = (d + 4) / 2 * 2.0 ** -23
        assert np.all(np.abs(got - ref[lower]) <= tol * ref[lower]), layout
