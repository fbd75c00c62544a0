"""An allocator that has no room for the float scan's scratch, or for the
index's row norms: the dense scans run in FP64 alone and return the same."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

N, NQ, D = 700, 900, 96


@pytest.fixture(scope="module")
def rr():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2502_13245_amd import rr as _rr
    _rr.lib()
    return _rr


def _limited(rr):
    class Limited(rr.TorchAllocator):
        """Refuses what `refuse` says; `sizes` lists every request."""

        def __init__(self, device=None):
            super().__init__(device)
            inner, self.sizes, self.refuse = self._alloc, [], lambda n: False

            def _alloc(nbytes, stream, ctx):
                self.sizes.append(int(nbytes))
                return None if self.refuse(int(nbytes)) else inner(nbytes, stream, ctx)
            self._inner, self._alloc = inner, rr.ALLOC_FN(_alloc)
            self.struct = rr.Allocator(self._alloc, self._free, None)
    return Limited


@pytest.fixture(scope="module")
def data():
    g = np.random.default_rng(3)
    x = g.standard_normal((N, D)).astype(np.float32)
    q = (x[g.integers(0, N, NQ)] + 0.1 * g.standard_normal((NQ, D))).astype(np.float32)
    E = ((x[None].astype(np.float64) - q[:, None].astype(np.float64)) ** 2).sum(2)
    s = np.sort(E.ravel())
    return x, q, E, 0.5 * (s[5000] + s[5001])


def _check(rr, ix, q, E, r):
    t = torch.from_numpy(q).cuda()
    off, ids, dd = rr.brute_force(ix, t, r).numpy()
    for i in range(len(q)):
        hit = np.flatnonzero(E[i] <= r)
        np.testing.assert_array_equal(np.sort(ids[off[i]:off[i + 1]]), hit)
        # float32 rounding of FP64 sums of 96 terms
        np.testing.assert_allclose(dd[off[i]:off[i + 1]], np.sort(E[i][hit]), rtol=2.0 ** -23)
    # FP64 sums from products: 2 (96 + 2) 2^-53 of the squared norms (below 400)
    np.testing.assert_allclose(rr.nn_dist(ix, t).cpu().numpy(), E.min(1), rtol=1e-12, atol=1e-11)


def test_no_room_for_the_scratch(rr, data, monkeypatch):
    x, q, E, r = data
    monkeypatch.setattr(rr, "TorchAllocator", _limited(rr))
    ix = rr.Index.from_graph(x, np.full((N, 1), -1, np.int32), 0).to_device("cuda:0")
    print("scan with and without scratch", flush=True)
    a = ix._alloc
    _check(rr, ix, q, E, r)
    # the scratch of 900 queries is 350 to 400 KB: refuse each call's first request
    big = max(a.sizes)
    rows = [s for s in a.sizes if 700_000 < s < 800_000]
    assert rows
    a.refuse = lambda n: n in (big, *rows)
    a.sizes.clear()
    _check(rr, ix, q, E, r)
    assert big in a.sizes and any(350_000 <= big - s <= 400_000 for s in a.sizes)


def test_no_room_for_the_norms(rr, data, monkeypatch):
    x, q, E, r = data
    cls = _limited(rr)

    class NoNorms(cls):
        def __init__(self, device=None):
            super().__init__(device)
            # (the graph, one id per point, asks for as much later on)
            self.refuse = lambda n: n == N * 4 and self.sizes.count(n) == 1
    monkeypatch.setattr(rr, "TorchAllocator", NoNorms)
    ix = rr.Index.from_graph(x, np.full((N, 1), -1, np.int32), 0).to_device("cuda:0")
    print("scan without norms", flush=True)
    assert N * 4 in ix._alloc.sizes
    _check(rr, ix, q, E, r)
