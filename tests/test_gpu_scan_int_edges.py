"""The integer range scan at the edges of its tiles (32, 64 and 128 points,
32 and 512 queries), of its row widths and of its bounds: whole numbers, so
every list equals the oracle's enumeration exactly."""
import numpy as np
import pytest

import oracle
from tests.gpu_common import flush_print

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def rr():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2502_13245_amd import rr as _rr
    _rr.lib()
    return _rr


def _rows(rng, n, d, dtype):
    i = np.iinfo(dtype)
    v = rng.integers(i.min, i.max + 1, size=(n, d)).astype(dtype)
    v[0], v[-1] = i.min, i.max  # the largest sums there are
    return v


@pytest.mark.parametrize("d", [1, 64, 65, 128, 192, 193, 256, 384, 385, 512])
@pytest.mark.parametrize("dtype,metric", [(np.uint8, "l2"), (np.int8, "l2"), (np.uint8, "ip"), (np.int8, "ip")])
def test_row_widths_and_odd_bounds(rr, d, dtype, metric):
    rng = np.random.default_rng(d)
    x, q = _rows(rng, 161, d, dtype), _rows(rng, 37, d, dtype)
    xi, qi = x.astype(np.int64), q.astype(np.int64)
    D = -(qi @ xi.T) if metric == "ip" else ((qi[:, None] - xi[None]) ** 2).sum(2)
    # a bound at a pair's distance, one below it, none and all: odd and even
    r = D[np.arange(37), rng.integers(0, 161, 37)].astype(np.float64)
    r[1::4] -= 1
    r[2::4] = [1e30, -1e30, -1.0][d % 3]
    flush_print(f"int scan d={d} {dtype.__name__} {metric}")
    ix = rr.Index.from_graph(x, np.full((161, 1), -1, np.int32), 0, metric=metric).to_device("cuda:0")
    off, ids, dd = rr.brute_force(ix, torch.from_numpy(q).cuda(), torch.from_numpy(r)).numpy()
    for i in range(37):
        hit = np.flatnonzero(D[i] <= r[i])
        hit = hit[np.lexsort((hit, D[i][hit]))]
        np.testing.assert_array_equal(ids[off[i]:off[i + 1]], hit)
        np.testing.assert_array_equal(dd[off[i]:off[i + 1]].astype(np.int64), D[i][hit])


@pytest.mark.parametrize("n", [1, 31, 32, 33, 127, 128, 129, 4097])
@pytest.mark.parametrize("nq", [1, 32, 33, 511, 513])
def test_tiles_of_points_and_queries(rr, n, nq):
    rng = np.random.default_rng(n * 1000 + nq)
    x = rng.integers(0, 256, size=(n, 100)).astype(np.uint8)
    q = rng.integers(0, 256, size=(nq, 100)).astype(np.uint8)
    r = float(np.quantile(oracle.pair_dists(x, q), 0.3))  # many hits in each tile
    flush_print(f"int scan n={n} nq={nq}")
    ix = rr.Index.from_graph(x, np.full((n, 1), -1, np.int32), 0).to_device("cuda:0")
    off, ids, dd = rr.brute_force(ix, torch.from_numpy(q).cuda(), r).numpy()
    o = oracle.brute_force(x, q, r)
    np.testing.assert_array_equal(off, o.offsets)
    np.testing.assert_array_equal(ids, o.ids)
    np.testing.assert_array_equal(dd.astype(np.int64), o.dists.astype(np.int64))
