"""edm_batched with rho = 0: whose decision a call takes.  The rows of X_cat
stand for point_off[S] only while they can: a longer buffer than the sets fill,
and a call that waits for the stream anyway, leave the look-up to the library."""
import numpy as np
import pytest

from paper_1308_1419_amd import synth, tdmap

S, D = 32, 3


def _batch(n, rows):
    torch = pytest.importorskip("torch")
    po = (torch.arange(S + 1) * n).cuda()
    oo = (torch.arange(S + 1) * (n * (n + 1) // 2)).cuda()
    X = torch.from_numpy(synth.uniform_points(rows, D, seed=n)).cuda()
    return X, po, oo, S * n * (n + 1) // 2


def test_least_cells():
    rng = np.random.default_rng(3)
    for _ in range(300):
        sizes = rng.integers(0, rng.integers(1, 60) + 1, size=rng.integers(1, 40))
        cells = int((sizes * (sizes + 1) // 2).sum())
        least = tdmap._least_cells(int(sizes.sum()), len(sizes))
        assert least <= cells
        if sizes.max() - sizes.min() <= 1:
            assert least == cells


@pytest.mark.gpu
def test_decision_of_the_right_class(monkeypatch):
    torch = pytest.importorskip("torch")
    assert torch.cuda.is_available()
    tdmap.tdmap_autotune_reset()
    asked = []
    call = tdmap.tdmap_edm_batched

    def spy(*args):
        asked.append(args[6])
        call(*args)

    monkeypatch.setattr(tdmap, "tdmap_edm_batched", spy)
    small, large = 12, 900
    want = {}
    for n in (small, large):
        X, po, oo, total = _batch(n, S * n)
        want[n] = tdmap.edm_batched(X, po, oo)  # waits: the library looks up and tunes
        tuned = tdmap.tdmap_tuned_rho(tdmap.OP_BATCHED, 0, n, D, S)
        assert asked.pop() == 0 and tuned in (1, 64, 128)
        out = torch.empty(total, device="cuda")
        tdmap.edm_batched(X, po, oo, out=out)  # the decision is there, the rows give its class
        assert asked.pop() == tuned
        assert torch.equal(out, want[n])
    # a buffer of the large sets' length that holds the small ones: not theirs
    X, po, oo, total = _batch(small, S * small)
    long = torch.cat([X, X.new_zeros(S * (large - small), D)])
    out = torch.empty(total, device="cuda")
    tdmap.edm_batched(long, po, oo, out=out)
    assert asked.pop() == 0
    assert torch.equal(out, want[small])


@pytest.mark.gpu
def test_negative_total_is_refused():
    # also with the class tuned: a call without `out` is looked up by the library,
    # which refuses before it launches anything
    torch = pytest.importorskip("torch")
    assert torch.cuda.is_available()
    X, po, oo, _ = _batch(12, S * 12)
    tdmap.edm_batched(X, po, oo)
    po[S] = -1
    with pytest.raises(tdmap.TdmapError) as e:
        tdmap.edm_batched(X, po, oo)
    assert e.value.status == tdmap.ERR_INVALID
