"""Nearest distances of more queries than fit one launch of a wave each
(2^26 waves are 2^32 threads)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def test_nearest_of_2_to_the_26_queries():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2502_13245_amd import rr
    n, nq = 64, (1 << 26) + 77
    if torch.cuda.mem_get_info()[0] < 40 << 30:
        pytest.skip("needs 40 GB")
    x = np.random.default_rng(1).standard_normal((n, 1)).astype(np.float32)
    ix = rr.Index.from_graph(x, np.full((n, 1), -1, np.int32), 0).to_device("cuda:0")
    q = torch.randn((nq, 1), generator=torch.Generator(device="cuda").manual_seed(2), device="cuda")
    print(f"{nq} queries", flush=True)
    nn = rr.nn_dist(ix, q)
    xs = torch.from_numpy(np.sort(x[:, 0])).cuda().double()
    for a in range(0, nq, 1 << 24):
        v = q[a:a + (1 << 24), 0].double()
        i = torch.searchsorted(xs, v).clamp(1, n - 1)
        # one square of an exact difference each: equal to the last bit
        assert torch.equal(nn[a:a + (1 << 24)], torch.minimum((v - xs[i - 1]) ** 2, (v - xs[i]) ** 2))
    del q, nn
    torch.cuda.empty_cache()
