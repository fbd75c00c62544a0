"""Float scans whose bfloat16 filter passes much (large radii, values far from
the origin, one long row): tiles with many candidates are decided by another
kernel.  Scans of fewer than 65,536 pairs decide every candidate by itself, so
a call in slices of that size is the reference, byte for byte; against plain
FP64 the tolerance is that of sums of d terms (below 4e-13 of their
magnitudes for d <= 900, 8e-13 for d <= 1,800)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def rr():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2502_13245_amd import rr as _rr
    _rr.lib()
    return _rr


def _index(rr, x, metric):
    return rr.Index.from_graph(x, np.full((len(x), 1), -1, np.int32), 0, metric=metric).to_device("cuda:0")


def _pairs(x, q, ip):
    x, q = x.astype(np.float64), q.astype(np.float64)
    D, M = np.empty((len(q), len(x))), np.empty((len(q), len(x)))
    for i in range(len(q)):
        t = x * q[i] if ip else (x - q[i]) ** 2
        D[i], M[i] = (-t.sum(1) if ip else t.sum(1)), np.abs(t).sum(1)
    return D, M


def _check(rr, x, q, r, metric, label):
    """r: a radius per query."""
    print(f"dense {label} {metric} n={len(x)} nq={len(q)} d={x.shape[1]}", flush=True)
    ix, t, rt = _index(rr, x, metric), torch.from_numpy(q).cuda(), torch.from_numpy(r)
    off, ids, dd = rr.brute_force(ix, t, rt).numpy()
    nn = rr.nn_dist(ix, t).cpu().numpy()
    step = 65535 // len(x)
    assert step >= 1 and len(x) * len(q) >= 65536
    for a in range(0, len(q), step):
        o2, i2, d2 = rr.brute_force(ix, t[a:a + step], rt[a:a + step]).numpy()
        b = min(a + step, len(q))
        np.testing.assert_array_equal(off[a:b + 1] - off[a], o2, err_msg=f"offsets from {a}")
        np.testing.assert_array_equal(ids[off[a]:off[b]], i2, err_msg=f"ids from {a}")
        np.testing.assert_array_equal(dd[off[a]:off[b]].view(np.uint32), d2.view(np.uint32), err_msg=f"dists from {a}")
        np.testing.assert_array_equal(nn[a:b], rr.nn_dist(ix, t[a:a + step]).cpu().numpy(), err_msg=f"nearest from {a}")
    D, M = _pairs(x, q, metric == "ip")
    tol = (4e-13 if x.shape[1] <= 900 else 8e-13) * M
    for i in range(len(q)):
        got = ids[off[i]:off[i + 1]]
        assert np.isin(np.flatnonzero(D[i] <= r[i] - tol[i]), got).all()
        assert (D[i][got] <= r[i] + tol[i][got]).all()
    return off, ids, dd


@pytest.mark.parametrize("metric", ["l2", "ip"])
# row splits of 4 to 64 lanes, 1 to 6 chunks a lane; odd counts of queries and points
@pytest.mark.parametrize("d,n,nq", [(16, 700, 129), (48, 641, 135), (30, 2049, 33), (90, 700, 101), (64, 1000, 71),
                                    (192, 999, 66), (128, 577, 127), (300, 700, 94), (256, 640, 104), (768, 1500, 50),
                                    (1000, 700, 97), (1536, 513, 129)])
def test_large_radii(rr, metric, d, n, nq):
    g = np.random.default_rng(d)
    x = g.standard_normal((n, d)).astype(np.float32)
    q = g.standard_normal((nq, d)).astype(np.float32)
    D, _ = _pairs(x, q, metric == "ip")
    r = np.quantile(D, 0.5, axis=1)
    r[::3] = np.quantile(D, 0.05, axis=1)[::3]  # some tiles are left to the other path
    r[1::16] = D.max() + 1
    r[2::16] = D.min() - 1
    _check(rr, x, q, r, metric, "radii")


@pytest.mark.parametrize("metric", ["l2", "ip"])
@pytest.mark.parametrize("kind", ["offset", "one long row", "two far groups"])
def test_wide_filter(rr, metric, kind):
    g = np.random.default_rng(5)
    x = g.standard_normal((1500, 96)).astype(np.float32)
    if kind == "offset":
        x += 100
    elif kind == "one long row":
        x[77] *= 1000
    else:
        x[700:] += 200
        x[:700] -= 200
    x[300:320] = x[3]
    q = np.concatenate([x[:50], x[1400:1450] + np.float32(0.1)])
    D, _ = _pairs(x, q, metric == "ip")
    off, ids, dd = _check(rr, x, q, np.quantile(D, 0.01, axis=1), metric, kind)
    if metric == "l2":
        assert (dd[off[:50]] == 0).all() and (dd[off[3]:off[3] + 21] == 0).all()


def test_not_finite_rows_in_whole_tiles(rr):
    g = np.random.default_rng(6)
    x = g.standard_normal((700, 40)).astype(np.float32)
    q = g.standard_normal((100, 40)).astype(np.float32)
    x[65, 3] = x[400, 0] = np.nan
    q[10], q[11, 4], q[12, 0] = 1e19, np.nan, np.inf
    r = np.full(100, 90.0)
    r[20:24] = [np.inf, 1e300, -1e300, 0.0]
    print("dense not finite", flush=True)
    ix, t, rt = _index(rr, x, "l2"), torch.from_numpy(q).cuda(), torch.from_numpy(r)
    got = rr.brute_force(ix, t, rt).numpy()
    D, _ = _pairs(x, q, False)
    for i in range(100):
        with np.errstate(invalid="ignore"):
            want = np.flatnonzero(D[i] <= r[i])
        assert set(got[1][got[0][i]:got[0][i + 1]]) == set(want), i
    nn = rr.nn_dist(ix, t).cpu().numpy()
    ok = np.setdiff1d(np.arange(100), [11, 12])
    np.testing.assert_allclose(nn[ok], np.nanmin(D[ok], axis=1), rtol=1e-12)
    assert np.isinf(nn[[11, 12]]).all()


def test_more_runs_than_are_kept(rr):
    """Dense and sparse tiles in turn, 262,144 runs where 131,072 are kept: the
    others' candidates are decided one by one."""
    n, nq, d = 1 << 20, 1024, 16
    g = torch.Generator(device="cuda").manual_seed(8)
    x = torch.randn((n, d), generator=g, device="cuda")
    x += torch.where(torch.arange(n, device="cuda") // 64 % 2 == 0, 300.0, -300.0)[:, None]
    q = torch.randn((nq, d), generator=g, device="cuda") + 300.0
    print("dense and sparse tiles in turn", flush=True)
    nn = rr.nn_dist(_index(rr, x.cpu().numpy(), "l2"), q)
    near = x.view(-1, 128, d)[:, :64].reshape(-1, d).double()
    for a in range(0, nq, 128):
        qa = q[a:a + 128].double()
        want = torch.full((len(qa),), float("inf"), dtype=torch.float64, device="cuda")
        for p in range(0, len(near), 1 << 14):
            s = torch.zeros((len(qa), min(1 << 14, len(near) - p)), dtype=torch.float64, device="cuda")
            for j in range(d):
                s += (qa[:, j:j + 1] - near[None, p:p + (1 << 14), j]) ** 2
            want = torch.minimum(want, s.min(1)[0])
        torch.testing.assert_close(nn[a:a + 128], want, rtol=1e-14, atol=0)
