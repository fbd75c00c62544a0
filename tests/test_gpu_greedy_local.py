"""Greedy expansion inside one workgroup: tasks around its limits (seeds,
list length, handing on to the level kernel, the set of a task handed on in
bitmaps or in the hash table) return the oracle's lists and counters."""
import numpy as np
import pytest

import oracle
from paper_2502_13245_amd import synth
from tests.gpu_common import check_greedy_edges, compare_exact, compare_float

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

N = 16000


@pytest.fixture(scope="module")
def rr():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2502_13245_amd import rr as _rr
    _rr.lib()
    return _rr


@pytest.fixture(scope="module")
def ball(rr):
    """Two tight clusters of 11K and 5K points: a query's list is long or short
    with its radius."""
    g = np.random.default_rng(11)
    x = np.empty((N, 16), np.uint8)
    for a, b, c in ((0, 11000, 60), (11000, N, 180)):
        x[a:b] = np.clip(np.rint(c + 8 * g.standard_normal((b - a, 16))), 0, 255)
    q = np.concatenate([x[g.integers(0, 11000, 6)], x[g.integers(11000, N, 6)]])
    adj, entry = oracle.build_vamana(x, 32, 48, 1.2, synth.permutation(N, 11))
    ix = rr.Index.from_graph(x, adj, entry).to_device("cuda:0")
    return x, q, adj, entry, ix, torch.from_numpy(q).cuda(), oracle.pair_dists(x, q)


def _radii(D, k):
    """Per query the distance of its k-th nearest point."""
    return np.sort(D, axis=1)[:, k - 1].astype(np.float64)


@pytest.mark.parametrize("nq", [1, 12])
@pytest.mark.parametrize("k", [40, 300, 1500, 4900, 10500])
def test_list_lengths(rr, ball, k, nq):
    x, q, adj, entry, ix, t, D = ball
    r = np.minimum(_radii(D, k), _radii(D, 4990) * 1.0001)[:nq] if k < 5000 else _radii(D, k)[:nq]
    print(f"lists of about {k}, {nq} queries", flush=True)
    o = oracle.range_search(x, adj, entry, q[:nq], r, mode=oracle.ADAPTIVE, beam=4)
    g = rr.range_search(ix, t[:nq], torch.from_numpy(r), mode="adaptive", beam=4, result_capacity=200_000)
    compare_exact(g, o, label=f"k={k}")
    check_greedy_edges(g, adj, label=f"k={k}")
    assert g.stats["expanded"].sum() > 0


@pytest.mark.parametrize("beam", [31, 32, 33, 64])
def test_seed_counts(rr, ball, beam):
    """|N| around the most seeds a workgroup takes; a mixed batch."""
    x, q, adj, entry, ix, t, D = ball
    r = _radii(D, 200)
    r[::3] = _radii(D, 2 * beam)[::3]
    print(f"seeds {beam}", flush=True)
    o = oracle.range_search(x, adj, entry, q, r, mode=oracle.ADAPTIVE, beam=beam, lam=0.5)
    g = rr.range_search(ix, t, torch.from_numpy(r), mode="adaptive", beam=beam, lam=0.5)
    compare_exact(g, o, label=f"beam={beam}")


@pytest.mark.parametrize("budget", ["0", "4096"])
def test_handed_on_sets(rr, ball, budget, monkeypatch):
    """Sets handed on in the hash table only, and for the first two tasks in
    bitmaps."""
    x, q, adj, entry, ix, t, D = ball
    monkeypatch.setenv("RR_BITMAP_BYTES", budget)
    r = _radii(D, 4500)
    print(f"bitmap budget {budget}", flush=True)
    o = oracle.range_search(x, adj, entry, q, r, mode=oracle.ADAPTIVE, beam=8)
    compare_exact(rr.range_search(ix, t, torch.from_numpy(r), mode="adaptive", beam=8,
                                  result_capacity=200_000), o, label="sets")


@pytest.mark.parametrize("cap", [100_000, 60_000, 9_000])
def test_capacities(rr, ball, cap):
    """Capacities down to the lists' total, also where the lists are too short
    for the task-local kernel; one entry less is reported."""
    x, q, adj, entry, ix, t, D = ball
    r = _radii(D, 700)
    print(f"capacity {cap}", flush=True)
    o = oracle.range_search(x, adj, entry, q, r, mode=oracle.ADAPTIVE, beam=4)
    compare_exact(rr.range_search(ix, t, torch.from_numpy(r), mode="adaptive", beam=4, result_capacity=cap), o,
                  label=f"cap={cap}")
    with pytest.raises(rr.RRError):
        rr.range_search(ix, t, torch.from_numpy(r), mode="adaptive", beam=4, result_capacity=2000)


@pytest.mark.parametrize("precision", ["exact", "bf16", "sq8"])
@pytest.mark.parametrize("d", [20, 400])
def test_float_passes(rr, precision, d):
    w = synth.latent_mixture_f32(4000, 40, d, 6, 0.1, 21)
    adj, entry = oracle.build_vamana(w.base, 24, 40, 1.2, synth.permutation(4000, 21))
    ix = rr.Index.from_graph(w.base, adj, entry).to_device("cuda:0")
    # (the percentile is one pair's distance, which float sums may put on
    # either side: just above it no pair is on the edge)
    r = oracle.percentile_radius(w.base, w.queries, 0.08) * (1 + 1e-9)
    code = {"exact": rr.EXACT, "bf16": rr.BF16_RECHECK, "sq8": rr.SQ8_RERANK}[precision]
    print(f"float {precision} d={d}", flush=True)
    g = rr.range_search(ix, torch.from_numpy(w.queries).cuda(), r, mode="adaptive", beam=6, precision=code)
    assert g.stats["expanded"].sum() > 5
    if precision == "exact":
        o = oracle.range_search(w.base, adj, entry, w.queries, r, mode=oracle.ADAPTIVE, beam=6)
        compare_float(g, o, r, label="exact")
        np.testing.assert_array_equal(g.stats["greedy_evals"], o.stats["greedy_evals"])
        return
    # every returned point is inside the ball at its FP64 distance (rounded to
    # float32), in order, and no point is returned twice
    off, ids, dd = g.numpy()
    for i in range(40):
        a = ids[off[i]:off[i + 1]]
        e = ((w.base[a].astype(np.float64) - w.queries[i].astype(np.float64)) ** 2).sum(1)
        assert len(np.unique(a)) == len(a) and (e <= r * (1 + 1e-12)).all()
        np.testing.assert_allclose(dd[off[i]:off[i + 1]], e, rtol=2.0 ** -23)
        assert (np.diff(dd[off[i]:off[i + 1]]) >= 0).all()
