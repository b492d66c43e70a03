"""Gram-form EDM with few features where many pairs are close relative to their
norms: a wave recomputes them in place instead of from its list.  A feature that
is 0 in every point adds an exact 0 to the products, the norms and the sums, so
33 features of which the last are 0, which always take the list, give the same
bits."""
import pytest

from paper_1308_1419_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_1308_1419_amd import tdmap  # noqa: E402


def _points(N, d, offset, seed):
    X, _ = synth.gaussian_with_near_duplicates(N, d, seed=seed, frac=0.02)
    return torch.from_numpy(X).cuda() + offset


@pytest.mark.parametrize("prec", ["bf16_gram", "bf16x3_gram"])
@pytest.mark.parametrize("offset", [0.0, 0.6, 3.0])
@pytest.mark.parametrize("N,d", [(2, 1), (33, 8), (300, 1), (300, 2), (300, 3), (600, 5), (257, 7), (1300, 8), (700, 4),
                                 (300, 9), (515, 12), (300, 15), (515, 16), (300, 17)])
def test_in_place_equals_list(N, d, offset, prec):
    assert torch.cuda.is_available()
    X = _points(N, d, offset, seed=N + d)
    P = torch.zeros((N, 33), device="cuda")
    P[:, :d] = X
    W = torch.full((N, d + 3), float("nan"), device="cuda")  # a pitch, 4 bytes past the base
    W[:, 1:d + 1] = X
    outs = []
    for x in (P, X, W[:, 1:d + 1]):
        for rho in (128, 256):
            buf = torch.full((N * (N + 1) // 2 + 64,), float("nan"), device="cuda")
            tdmap.edm(x, layout="packed", rho=rho, precision=prec, out=buf)
            _, count = tdmap.gram_recompute_count(x, prec, rho=rho)
            outs.append((buf.view(torch.int32), int(count)))
    for bits, count in outs[1:]:
        assert torch.equal(bits, outs[0][0]) and count == outs[0][1]
    if offset == 3.0 and N > 2:
        assert outs[0][1] > 0.8 * N * (N + 1) / 2


def test_close_pairs_of_few_features():
    # every pair recomputed at two features against hardly one at 16: 9.8 times
    # as long from the list, 2.1 in place.  At most 4.
    assert torch.cuda.is_available()
    N = 12000
    out = torch.empty(N * (N + 1) // 2, device="cuda")
    X = [torch.randn((N, 16), device="cuda"), torch.randn((N, 2), device="cuda") + 3.0]
    ws = torch.empty(tdmap.tdmap_workspace_size(tdmap.OP_EDM, N, 16, 0, 256, tdmap.BF16_GRAM),
                     dtype=torch.uint8, device="cuda")
    times = ([], [])
    for _ in range(7):
        for x, t in zip(X, times):
            begin, end = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            begin.record()
            for _ in range(20):
                tdmap.edm(x, layout="packed", rho=256, precision="bf16_gram", out=out, workspace=ws)
            end.record()
            end.synchronize()
            t.append(begin.elapsed_time(end))
    assert min(times[1][1:]) <= 4 * min(times[0][1:])
