"""The binding issues its work on torch's current stream, and takes the batched
tuner's decision without reading the offsets back: a call on a stream that is
held back by other work must not run ahead of it, and must not wait for it."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_1308_1419_amd import tdmap  # noqa: E402


def test_calls_follow_the_current_stream():
    assert torch.cuda.is_available()
    S, n = 32, 40
    X0 = torch.rand(S * n, 3, device="cuda")
    po = torch.arange(S + 1, device="cuda") * n
    oo = torch.arange(S + 1, device="cuda") * (n * (n + 1) // 2)
    want = [tdmap.edm(X0), tdmap.edm_batched(X0, po, oo)]  # tunes both
    dD = torch.rand_like(want[1])
    want.append(tdmap.edm_backward(X0[:n], dD))
    torch.cuda.synchronize()
    busy = torch.rand(4096, 4096, device="cuda")
    X = torch.zeros_like(X0)
    out = torch.empty(S * n * (n + 1) // 2, device="cuda")
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    done = torch.cuda.Event()
    with torch.cuda.stream(side):
        for _ in range(40):
            busy = busy @ busy * 1e-4
        X.copy_(X0)  # the points arrive behind the products
        got = [tdmap.edm(X), tdmap.edm_batched(X, po, oo, out=out), tdmap.edm_backward(X[:n], dD)]
        done.record()
    assert not done.query(), "a call waited for the stream"
    side.synchronize()
    low = torch.ones_like(want[0], dtype=torch.bool).tril()
    assert torch.equal(got[0][low], want[0][low])
    assert torch.equal(got[1], want[1]) and torch.equal(got[2], want[2])
