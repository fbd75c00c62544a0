"""The beam of one wave at the widths where its form changes (keys in the
lanes up to 64, an LDS array with late keys in the lanes above), with a seen
cache of 64 ids that forgets nearly everything: results and visits are the
oracle's."""
import numpy as np
import pytest

import oracle
from paper_2502_13245_amd import synth
from tests.gpu_common import compare_exact, compare_float

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

N, NQ = 3000, 60


@pytest.fixture(scope="module")
def rr():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2502_13245_amd import rr as _rr
    _rr.lib()
    return _rr


@pytest.fixture(scope="module")
def u8(rr):
    w = synth.latent_mixture_u8(N, NQ, 24, 12, 25.0, 3)
    adj, entry = oracle.build_vamana(w.base, 40, 64, 1.2, synth.permutation(N, 3))
    ix = rr.Index.from_graph(w.base, adj, entry).to_device("cuda:0")
    return w, adj, entry, ix, torch.from_numpy(w.queries).cuda(), oracle.percentile_radius(w.base, w.queries, 0.02)


@pytest.fixture(scope="module")
def f32(rr):
    w = synth.latent_mixture_f32(N, NQ, 20, 12, 0.35, 4)
    adj, entry = oracle.build_vamana(w.base, 40, 64, 1.2, synth.permutation(N, 4))
    ix = rr.Index.from_graph(w.base, adj, entry).to_device("cuda:0")
    return w, adj, entry, ix, torch.from_numpy(w.queries).cuda(), oracle.percentile_radius(w.base, w.queries, 0.02)


WIDTHS = [1, 2, 23, 24, 25, 63, 64, 65, 66, 127, 128, 129, 255, 700, 3000]


@pytest.mark.parametrize("slots", [64, 0])
@pytest.mark.parametrize("beam", WIDTHS)
def test_plain_widths_u8(rr, u8, beam, slots):
    w, adj, entry, ix, q, r = u8
    print(f"beam {beam} slots {slots}", flush=True)
    o = oracle.range_search(w.base, adj, entry, w.queries, r, mode=oracle.PLAIN, beam=beam)
    for wpg in (1, 4):
        g = rr.range_search(ix, q, r, mode="plain", beam=beam, cache_slots=slots, waves_per_group=wpg)
        compare_exact(g, o, check_evals=slots == 0, label=f"b={beam}")
        assert slots == 0 or beam < 24 or g.stats["cache_overflow"].any()


@pytest.mark.parametrize("beam", [1, 24, 64, 65, 129, 700])
def test_widths_f32(rr, f32, beam):
    w, adj, entry, ix, q, r = f32
    print(f"float beam {beam}", flush=True)
    for mode, om in (("plain", oracle.PLAIN), ("adaptive", oracle.ADAPTIVE)):
        o = oracle.range_search(w.base, adj, entry, w.queries, r, mode=om, beam=beam)
        g = rr.range_search(ix, q, r, mode=mode, beam=beam, cache_slots=64)
        compare_float(g, o, r, label=f"{mode} b={beam}")
        np.testing.assert_array_equal(g.stats["visits"], o.stats["visits"])


@pytest.mark.parametrize("beam,top,es", [(1, 64, False), (3, 200, False), (60, 130, True), (64, 1000, False)])
def test_doubling_across_the_forms(rr, u8, beam, top, es):
    w, adj, entry, ix, q, r = u8
    kw = dict(beam=beam, max_beam=top, es_enable=es, es_visit_limit=4, es_radius=2 * r)
    print(f"doubling {beam}..{top}", flush=True)
    o = oracle.range_search(w.base, adj, entry, w.queries, r, mode=oracle.DOUBLING, **kw)
    g = rr.range_search(ix, q, r, mode="doubling", cache_slots=64, **kw)
    off, ids, dd = g.numpy()
    np.testing.assert_array_equal(off, o.offsets)
    np.testing.assert_array_equal(ids, o.ids)
    np.testing.assert_array_equal(dd.astype(np.int64), o.dists.astype(np.int64))
    for k in ("visits", "rounds", "final_beam", "truncated"):
        np.testing.assert_array_equal(g.stats[k], o.stats[k], err_msg=k)


@pytest.mark.parametrize("beam", [24, 64, 65, 200])
def test_resumed_after_every_visit(rr, u8, beam):
    """A served search suspended after each visit keeps its beam."""
    w, adj, entry, ix, q, r = u8
    print(f"resumed beam {beam}", flush=True)
    o = oracle.range_search(w.base, adj, entry, w.queries, r, mode=oracle.PLAIN, beam=beam)
    with rr.Server(ix, rr.search_params(mode="plain", beam=beam, cache_slots=64), slots=NQ, step_budget=1) as s:
        for i in range(NQ):
            assert s.submit(w.queries[i], r, i)
        s.drain(100.0)
        done = {c.tag: c for c in s.poll()}
        for i in range(NQ):
            ids, dd = s.result(i)
            oi, od = o.query(i)
            np.testing.assert_array_equal(ids, oi)
            np.testing.assert_array_equal(dd.astype(np.int64), np.asarray(od).astype(np.int64))
            assert done[i].stats.visits == o.stats["visits"][i]
