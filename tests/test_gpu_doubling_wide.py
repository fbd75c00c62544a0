"""Doubling rounds wider than 4,096 keys whose width is no multiple of 64: the
last round's beam is full, and every list is the oracle's."""
import numpy as np
import pytest

import oracle
from paper_2502_13245_amd import synth
from tests.gpu_common import compare_float

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

N, NQ = 12000, 4


@pytest.fixture(scope="module")
def rr():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2502_13245_amd import rr as _rr
    _rr.lib()
    return _rr


@pytest.fixture(scope="module", params=["u8", "f32"])
def ball(rr, request):
    """One cluster, so that a ball of any size is connected."""
    g = np.random.default_rng(31)
    x = 120 + 20 * g.standard_normal((N, 16))
    x = np.clip(np.rint(x), 0, 255).astype(np.uint8) if request.param == "u8" else x.astype(np.float32)
    q = x[g.integers(0, N, NQ)]
    adj, entry = oracle.build_vamana(x, 32, 48, 1.2, synth.permutation(N, 31))
    ix = rr.Index.from_graph(x, adj, entry).to_device("cuda:0")
    D = ((x[None].astype(np.float64) - q[:, None].astype(np.float64)) ** 2).sum(2)
    return x, q, adj, entry, ix, np.sort(D, axis=1)


@pytest.mark.parametrize("fill", [0.6, 1.1])
@pytest.mark.parametrize("beam,top", [(129, 4096), (750, 4096), (1500, 4096), (1500, 6000), (2050, 4100), (2100, 8400)])
def test_last_round_is_full(rr, ball, beam, top, fill):
    x, q, adj, entry, ix, D = ball
    last = beam
    while last < top:
        last *= 2
    assert last > 4096 and last % 64 != 0
    if x.dtype == np.float32 and last > 6448:
        with pytest.raises(rr.RRError):
            rr.range_search(ix, torch.from_numpy(q).cuda(), 1.0, mode="doubling", beam=beam, max_beam=top)
        return
    # halfway between two neighbouring distances where they differ
    k = int(fill * last)
    r = 0.5 * (D[:, k - 1] + D[:, k])
    print(f"doubling {x.dtype} {beam}..{top} ({last}) fill {fill}", flush=True)
    kw = dict(beam=beam, max_beam=top)
    o = oracle.range_search(x, adj, entry, q, r, mode=oracle.DOUBLING, **kw)
    assert (o.stats["final_beam"] == last).all()
    g = rr.range_search(ix, torch.from_numpy(q).cuda(), torch.from_numpy(r), mode="doubling",
                        result_capacity=NQ * 2 * N, **kw)
    for name in ("visits", "rounds", "final_beam", "truncated", "count"):
        np.testing.assert_array_equal(g.stats[name], o.stats[name], err_msg=name)
    if x.dtype == np.uint8:
        off, ids, dd = g.numpy()
        np.testing.assert_array_equal(off, o.offsets)
        np.testing.assert_array_equal(ids, o.ids)
        np.testing.assert_array_equal(dd.astype(np.int64), o.dists.astype(np.int64))
    else:
        compare_float(g, o, r, label=f"{beam}..{top}")
        np.testing.assert_array_equal(g.numpy()[0], o.offsets)
