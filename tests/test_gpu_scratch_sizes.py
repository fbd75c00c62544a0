"""What a search needs beside its results stays within what callers size
their scratch, capacities and budgets by: requests of
rr_range_search_noalloc that just fit, and the slots of a serving budget."""
import re

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

N = 500


@pytest.fixture(scope="module")
def rr():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2502_13245_amd import rr as _rr
    _rr.lib()
    return _rr


@pytest.fixture(scope="module", params=[np.uint8, np.float32])
def ctx(rr, request):
    x = np.random.default_rng(0).integers(0, 256, size=(N, 16)).astype(request.param)
    adj = np.array([[(i + j + 1) % N for j in range(8)] for i in range(N)], np.int32)
    return x, rr.Index.from_graph(x, adj, 0).to_device("cuda:0")


# bytes of scratch for a result capacity of 2^23 (integer data, float data)
NEED = {(1, 8): (872461312, 1006679040), (1000, 8): (873023232, 1007368960), (50000, 2): (888757760, 1024574976)}


@pytest.mark.parametrize("nq,beam", list(NEED))
def test_noalloc_needs_no_more(rr, ctx, nq, beam):
    x, ix = ctx
    print(f"scratch of {nq} queries, beam {beam}, {x.dtype}", flush=True)
    q = torch.from_numpy(x[np.arange(nq) % N]).cuda()
    with pytest.raises(rr.RRError) as e:
        rr.range_search_noalloc(ix, q, 1.0, capacity=16, mode="adaptive", beam=beam, result_capacity=1 << 23)
    assert int(re.search(r"need (\d+) bytes", str(e.value)).group(1)) <= NEED[nq, beam][x.dtype == np.float32]


# slots that a budget holds at beam 8 and a result capacity of 100,000
SLOTS = {1 << 24: (16358, 11664), 3 << 24: (59488, 46836)}


@pytest.mark.parametrize("budget", list(SLOTS))
def test_a_budget_holds_as_many_slots(rr, ctx, budget):
    x, ix = ctx
    print(f"slots of {budget} bytes, {x.dtype}", flush=True)
    with rr.Server(ix, rr.search_params(mode="adaptive", beam=8), slots=0, hbm_budget=budget,
                   result_capacity=100_000) as s:
        info = s.info()
    assert info["slots"] >= SLOTS[budget][x.dtype == np.float32] and info["device_bytes"] <= budget
