"""The greedy phase's levels: their points add up to the phase's items and
their times lie within the phase, with tasks expanded inside one workgroup,
left to the level kernel from their seeds on, handed on to it, and without the
task-local kernel (lists too short for it)."""
import numpy as np
import pytest

import oracle
from paper_2502_13245_amd import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

N, NQ = 12000, 8


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2502_13245_amd import rr
    rr.lib()
    g = np.random.default_rng(41)
    x = np.clip(np.rint(100 + 12 * g.standard_normal((N, 16))), 0, 255).astype(np.uint8)
    q = x[g.integers(0, N, NQ)]
    adj, entry = oracle.build_vamana(x, 32, 48, 1.2, synth.permutation(N, 41))
    ix = rr.Index.from_graph(x, adj, entry).to_device("cuda:0")
    return rr, ix, torch.from_numpy(q).cuda(), np.sort(oracle.pair_dists(x, q), axis=1)


# k-th nearest as the radius, beam, result capacity; levels that take part
@pytest.mark.parametrize("k,beam,cap,levels", [(200, 4, 100_000, "local"), (200, 64, 100_000, "left"),
                                               (9000, 4, 200_000, "handed on"), (200, 4, 3_000, "level kernel"),
                                               (1, 4, 100_000, "none")])
def test_times_lie_within_the_phase(ctx, k, beam, cap, levels):
    rr, ix, q, D = ctx
    r = D[:, k - 1].astype(np.float64) if k > 1 else -np.ones(NQ)
    print(f"levels: {levels}", flush=True)
    for _ in range(2):
        g = rr.range_search(ix, q, torch.from_numpy(r), mode="adaptive", beam=beam, result_capacity=cap, timing=True)
    b = g.batch
    lv = b["levels"]
    assert len(lv) == min(b["greedy_levels"], 64)
    if levels == "none":
        assert not lv
        return
    assert sum(x["items"] for x in lv) == b["greedy_items"] == int(g.stats["greedy_visits"].sum())
    # what each case is for
    handed = sum(x["items"] for x in lv[2:])
    assert {"local": len(lv) == 2 and lv[1]["items"] > 0, "left": len(lv) > 2 and lv[1]["items"] == 0,
            "handed on": lv[1]["items"] > 0 and handed > 0, "level kernel": len(lv) > 3}[levels]
    times = [x[t] for x in lv for t in ("expand_ms", "regroup_ms")]
    assert all(0.0 <= t <= b["greedy_kernel_ms"] for t in times)
    # the profile's entries are rounded to 0.1 us; its clock ticks at 100 MHz
    assert 0.0 < sum(times) <= b["greedy_kernel_ms"] + 0.0002 * len(times)
    # levels that expanded points took time
    for i, x in enumerate(lv):
        if x["items"] and not (i == 0 and levels in ("local", "handed on")):
            assert x["expand_ms"] > 0.0
