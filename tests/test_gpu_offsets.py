"""Result offsets at the edges of their scan: its workgroup's tile (8,192
counts), the largest batch that one workgroup scans (16,384) and the one
above; whole numbers, equal to the running sums."""
import numpy as np
import pytest

from tests.gpu_common import flush_print

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("nq", [1, 7, 8, 63, 511, 513, 8191, 8192, 8193, 16383, 16384, 16385, 24577])
def test_offsets_are_the_running_sums(nq):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2502_13245_amd import rr
    rng = np.random.default_rng(nq)
    x = rng.integers(0, 256, size=(9, 4)).astype(np.uint8)
    q = rng.integers(0, 256, size=(nq, 4)).astype(np.uint8)
    D = ((q[:, None].astype(np.int64) - x[None].astype(np.int64)) ** 2).sum(2)
    r = rng.integers(-1, int(D.max()) + 1, size=nq).astype(np.float64)
    flush_print(f"offsets nq={nq}")
    ix = rr.Index.from_graph(x, np.full((9, 1), -1, np.int32), 0).to_device("cuda:0")
    off, ids, dd = rr.brute_force(ix, torch.from_numpy(q).cuda(), torch.from_numpy(r)).numpy()
    cnt = (D <= r[:, None]).sum(1)
    np.testing.assert_array_equal(off, np.concatenate([[0], np.cumsum(cnt)]))
    np.testing.assert_array_equal(dd.astype(np.int64), D[np.repeat(np.arange(nq), cnt), ids])
