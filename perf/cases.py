"""The workloads that timings of this library are taken on.

A case is a dict of plain values: the index (element type, metric, n, d, R),
the operation, and its options.  `prepare` makes the seeded queries (and
per-query radii) of one call; the index is the handle a program keeps between
calls, made from the case's own values and held here for the next
preparation.  Base points and queries follow the mixtures of the synthetic
workloads (centres on a 16-dimensional sheet, a 10-dimensional basis per
cluster, Zipf cluster sizes, a tenth of the clusters near-duplicate groups),
drawn on the GPU; the graph links each point to its nearest neighbours in two
cluster-wise orders, to members of the nearest clusters and to a few random
points, so that a beam search can walk it.  Small indices get the library's
own Vamana graph.  Everything that the graph depends on is integer arithmetic
or elementwise, so every process makes the same index.
"""
from __future__ import annotations

import math
from collections import OrderedDict

import numpy as np
import torch

from paper_2502_13245_amd import rr

NP = {"u8": np.uint8, "i8": np.int8, "f32": np.float32}
ES = {"u8": 1, "i8": 1, "f32": 4}
PRECISION = {"exact": rr.EXACT, "bf16": rr.BF16_RECHECK, "sq8": rr.SQ8_RERANK}
DEV = "cuda:0"

_U8 = dict(dtype="u8", metric="l2", n=1_000_000, d=128, R=64)
_F32 = dict(dtype="f32", metric="l2", n=1_000_000, d=96, R=64)
_WIDE = dict(dtype="f32", metric="ip", n=100_000, d=768, R=32)


def listed():
    return [
        # one lookup against a small collection with default options, counters
        # included: the latency of the smallest call
        dict(name="one-query", op="search", dtype="u8", metric="l2", n=10_000, d=128, R=32, nq=1,
             mode="adaptive", beam=32, nonempty=0.9, stats=True),
        # an interactive batch against a million points, default beam
        dict(name="batch-64", op="search", **_U8, nq=64, mode="adaptive", beam=32, nonempty=0.25),
        # the headline: 10,000 queries, half of them empty, narrow beam and early stop
        dict(name="adaptive-10k", op="search", **_U8, nq=10_000, mode="adaptive", beam=8, es=True,
             vl=20, esr=15.0, nonempty=0.5, cache_slots=1024, waves=4),
        # the plain wide beam that range search without expansion needs for recall
        dict(name="plain-wide", op="search", **_U8, nq=1_000, mode="plain", beam=1024, nonempty=0.25),
        # Algorithm 3, rounds up to a beam of 4,096
        dict(name="doubling", op="search", **_U8, nq=1_000, mode="doubling", beam=16, max_beam=4096,
             nonempty=0.25),
        # float embeddings, bfloat16 first pass, heavy result lists
        dict(name="embed-bf16", op="search", **_F32, nq=10_000, mode="adaptive", beam=4, es=True,
             vl=10, esr=1.0, nonempty=0.85, precision="bf16", cap=1 << 24),
        # the same collection in exact arithmetic, fewer queries, a wider beam
        dict(name="embed-exact", op="search", **_F32, nq=2_500, mode="adaptive", beam=16, nonempty=0.5,
             cap=1 << 23),
        # text embeddings under the inner product, 8-bit first pass
        dict(name="text-sq8-ip", op="search", **_WIDE, nq=1_000, mode="adaptive", beam=32,
             nonempty=0.5, precision="sq8", cap=1 << 22),
        # a larger int8 collection (rows of 100 values), a large batch; above
        # four million points the membership set is the hash table
        dict(name="large-i8", op="search", dtype="i8", metric="l2", n=4_500_000, d=100, R=32,
             nq=20_000, mode="adaptive", beam=16, es=True, vl=20, esr=15.0, nonempty=0.25, cap=1 << 23),
        # exact ground truth by the dense scan, integer and float
        dict(name="scan-u8", op="scan", **_U8, nq=10_000, nonempty=0.25),
        dict(name="scan-f32", op="scan", **_F32, nq=2_000, nonempty=0.25),
        # a burst of requests through the serving loop
        dict(name="serve-burst", op="serve", **_WIDE, nq=32, mode="adaptive", beam=8, nonempty=0.5,
             precision="bf16", slots=256, cap=1 << 21),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges: element types, metrics, ragged widths,
    batch sizes from one query up, every mode, precision and dense scan."""
    op = rng.choice(["search"] * 7 + ["scan", "nn", "radius"])
    dtype = rng.choice(["u8", "i8", "f32"])
    d = _log_int(rng, 7, 768 if dtype == "f32" else 500)
    n = _log_int(rng, 3_000, min(300_000, 60_000_000 // d))
    c = dict(op=op, dtype=dtype, metric=rng.choice(["l2", "l2", "ip"]), n=n, d=d,
             R=rng.choice([16, 24, 32, 48, 64]), nonempty=rng.choice([0.25, 0.5, 0.85]))
    if op != "search":
        # the dense scans: products bounded by the listed ones
        top = min(5_000, int((4e10 if dtype == "f32" else 4e11) / (n * d)))
        c["nq"] = _log_int(rng, 1, max(1, top if op != "radius" else min(top, 100_000_000 // n)))
        if op == "radius":
            c["p"] = rng.choice([0.0005, 0.001, 0.01])
        return c
    mode = rng.choice(["adaptive"] * 4 + ["plain", "es", "doubling"])
    c["mode"] = mode
    if mode == "doubling":
        c.update(nq=_log_int(rng, 1, 500), beam=rng.choice([2, 4, 8, 20]), max_beam=rng.choice([64, 300, 1024]))
    elif mode == "adaptive":
        c.update(nq=_log_int(rng, 1, 6_000), beam=_log_int(rng, 2, 100))
    else:
        beam = _log_int(rng, 8, 1024)
        c.update(beam=beam, nq=_log_int(rng, 1, max(1, min(6_000, 500_000 // beam))))
    if mode == "es" or (mode != "plain" and rng.random() < 0.5):
        # the multiple of the radius is of use for a distance; inner products stop at the radius
        c.update(es=True, vl=rng.choice([2, 5, 20]),
                 esr=1.0 if c["metric"] == "ip" else rng.choice([1.0, 4.0, 15.0]))
    if dtype == "f32" and mode != "doubling":
        c["precision"] = rng.choice(["exact", "bf16", "sq8"])
    if rng.random() < 0.3:
        c["radii"] = True  # a radius per query
    if rng.random() < 0.2:
        c["most"] = rng.choice([10, 100, 1000])  # max_results_per_query
    c["cap"] = 1 << 23 if mode == "adaptive" or mode == "doubling" else 0
    return c


# ---------------------------------------------------------------------------
# data and graphs
# ---------------------------------------------------------------------------

class _Mixture:
    """The clusters of one collection; draws points of it on the GPU."""

    def __init__(self, dtype, n, d, unit):
        self.dtype, self.d, self.unit = dtype, d, unit
        g = torch.Generator(device=DEV).manual_seed(1000 + d)
        k = self.k = int(min(4000, max(16, n // 1000)))
        std, sigma, noise, dense = {"u8": (40.0, 25.0, 4.0, 6.0), "i8": (30.0, 20.0, 3.0, 5.0),
                                    "f32": (1.0, 0.35, 0.05, 0.1)}[dtype]
        self.mid, self.noise = (127.5 if dtype == "u8" else 0.0), noise

        def normal(*shape):
            return torch.randn(shape, generator=g, device=DEV)

        A, u = normal(16, d) * (std / 4.0), normal(k, 16)
        c = torch.zeros(k, d, device=DEV)
        for j in range(16):
            c += u[:, j:j + 1] * A[j]
        self.centers = c + self.mid
        spread = torch.rand(k, generator=g, device=DEV) * 2 - 1
        self.scale = sigma * torch.exp(0.35 * spread)
        # near-duplicate groups: a tenth of the clusters, the very largest not among them
        near = torch.rand(k, generator=g, device=DEV) < 0.1
        near[:8] = False
        self.scale[near] = dense * torch.exp(0.5 * spread[near])
        self.basis = normal(k, 10, d) / math.sqrt(10.0)
        w = 1.0 / np.arange(1, k + 1)
        self.cdf = torch.from_numpy(np.cumsum(w / w.sum())).to(DEV)

    def labels(self, m, g):
        u = torch.rand(m, generator=g, device=DEV, dtype=torch.float64)
        return torch.searchsorted(self.cdf, u).clamp_(max=self.k - 1)

    def points(self, lab, g):
        out = torch.empty(len(lab), self.d, device=DEV,
                          dtype={"u8": torch.uint8, "i8": torch.int8, "f32": torch.float32}[self.dtype])
        step = max(1, (1 << 27) // self.d)
        for a in range(0, len(lab), step):
            lb = lab[a:a + step]
            z = torch.randn((len(lb), 10), generator=g, device=DEV) * self.scale[lb][:, None]
            v = self.centers[lb]
            for j in range(10):
                v = v + z[:, j:j + 1] * self.basis[:, j][lb]
            v += self.noise * torch.randn((len(lb), self.d), generator=g, device=DEV)
            if self.dtype == "u8":
                v = v.round_().clamp_(0, 255)
            elif self.dtype == "i8":
                v = v.round_().clamp_(-128, 127)
            elif self.unit:
                v = v / v.double().square().sum(1, keepdim=True).sqrt().float()
            out[a:a + step] = v.to(out.dtype)
        return out


def _whole(x):
    """The points as whole numbers in [-128, 127] (float32), for the graph."""
    if x.dtype == torch.uint8:
        return x.float() - 128
    if x.dtype == torch.int8:
        return x.float()
    return (x * (127.0 / float(x.abs().max()))).round_()


def _graph(x, lab, mix, R, g):
    """R-out graph over points sorted by cluster: rows of distinct ids, -1 at
    the end.  Two passes of nearest neighbours inside windows of 1,024 points
    (ordered within a cluster by a random projection), then random members of
    the point's own cluster, then members of the nearest clusters, then random
    points."""
    n, d = x.shape
    W = 1024
    own, near, far = R // 8, R // 4, R // 4
    knn = (R - own - near - far) // 2
    w = _whole(x)
    shift = max(0, int(math.ceil(math.log2(max(1.0, 4.0 * d * 128 * 128)))) - 21)
    parts = []
    for p in range(2):
        sign = (torch.randint(0, 2, (d,), generator=g, device=DEV) * 2 - 1).float()
        proj = torch.empty(n, device=DEV, dtype=torch.float64)
        for a in range(0, n, 1 << 18):
            proj[a:a + (1 << 18)] = (w[a:a + (1 << 18)] * sign).double().sum(1)
        order = torch.sort(lab.double() * 1e9 + proj, stable=True)[1]
        got = torch.full((n, knn), -1, dtype=torch.int64, device=DEV)
        for a in range(0, n, W * 64):
            o = order[a:a + W * 64]
            m = len(o)
            o = torch.cat([o, o.new_full(((-m) % W,), -1)]).view(-1, W)
            v = torch.where((o >= 0)[..., None], w[o.clamp(min=0)], torch.full((), 1e4, device=DEV))
            sq = (v * v).sum(2)
            d2 = sq[:, :, None] + sq[:, None, :] - 2 * torch.bmm(v, v.transpose(1, 2).contiguous())
            # unique keys (distance, position), so that ties have one order
            key = (d2.clamp_(0, 2.0 ** 40).to(torch.int64) >> shift).clamp_(max=(1 << 21) - 2).to(torch.int32)
            key.masked_fill_((o < 0)[:, None, :], (1 << 21) - 1)
            key.diagonal(dim1=1, dim2=2).fill_((1 << 21) - 1)
            key = key * W + torch.arange(W, device=DEV, dtype=torch.int32)
            val, idx = torch.topk(key, knn, dim=2, largest=False)
            ids = torch.gather(o[:, None, :].expand(-1, W, -1), 2, idx)
            ids = torch.where((val >> 10) >= (1 << 21) - 1, torch.full_like(ids, -1), ids)
            got[o.reshape(-1)[:m]] = ids.reshape(-1, knn)[:m]
        parts.append(got)
    # cluster c's points are [first[c], first[c + 1]) in the sorted numbering
    first = torch.searchsorted(lab, torch.arange(mix.k + 1, device=DEV))
    size = first[1:] - first[:-1]
    c = (mix.centers - mix.mid)
    c = (c * (64.0 / float(c.abs().max()))).round_()
    sq = (c * c).sum(1)
    cd = (sq[:, None] + sq[None, :] - 2 * (c @ c.T.contiguous())).to(torch.int64) * 8192
    cd += torch.arange(mix.k, device=DEV)
    cd[:, size == 0] = 1 << 60
    nc = torch.topk(cd, min(1 + near, mix.k), dim=1, largest=False)[1][lab]
    nc = torch.cat([nc[:, :1].expand(-1, own), nc[:, 1:]], 1)  # the nearest is its own
    u = torch.rand((n, nc.shape[1]), generator=g, device=DEV)
    parts.append(first[nc] + torch.minimum((u * size[nc]).long(), (size[nc] - 1).clamp(min=0)))
    parts.append(torch.randint(0, n, (n, far), generator=g, device=DEV))
    adj = torch.cat(parts, 1)
    adj[adj == torch.arange(n, device=DEV)[:, None]] = -1
    adj = torch.where(adj < 0, torch.full_like(adj, n), adj).sort(1)[0]
    adj[:, 1:][adj[:, 1:] == adj[:, :-1]] = n
    return adj.sort(1)[0]


def _pair_min(x, q, ip):
    """The smallest distance of each query, in 64 bits (exact for whole numbers)."""
    q = q.double()
    best = torch.full((len(q),), math.inf, dtype=torch.float64, device=DEV)
    step = max(1, (1 << 27) // max(len(q), x.shape[1]))
    for a in range(0, len(x), step):
        v = x[a:a + step].double()
        dot = q @ v.T.contiguous()
        dd = -dot if ip else q.square().sum(1)[:, None] + v.square().sum(1)[None] - 2 * dot
        best = torch.minimum(best, dd.min(1)[0])
    return best


_indices: OrderedDict = OrderedDict()
_HELD = 8


class _Collection:
    def __init__(self, dtype, metric, n, d, R):
        g = torch.Generator(device=DEV).manual_seed(n)
        self.mix = mix = _Mixture(dtype, n, d, unit=True)
        lab = mix.labels(n, g).sort()[0]
        x = mix.points(lab, g)
        self.ip = metric == "ip"
        perm = torch.randperm(n, generator=torch.Generator().manual_seed(n)).to(DEV)  # new number of point i
        base = torch.empty_like(x)
        base[perm] = x
        if n <= 20_000 and d <= 200:
            self.index = rr.Index.build(base.cpu().numpy(), R=R, L=2 * R, passes=1, threads=8, metric=metric)
        else:
            adj = _graph(x, lab, mix, R, g)
            new = torch.full((n, R), -1, dtype=torch.int32, device=DEV)
            new[perm, :adj.shape[1]] = torch.where(adj < n, perm[adj.clamp(max=n - 1)], torch.full_like(adj, -1)).int()
            w = _whole(base)
            off = (w - w.double().mean(0).round().float()).square().sum(1).double() * n
            entry = int((off + torch.arange(n, device=DEV)).argmin())
            self.index = rr.Index.from_graph(base.cpu().numpy(), new.cpu().numpy(), entry, metric=metric)
        self.index.to_device(DEV)
        # the radii of the collection: quantiles of the distance to the nearest point
        nn = _pair_min(base, self.queries(512, 77), self.ip).sort()[0].cpu().numpy()
        self.radii = {f: float("%.5g" % nn[int(f * 511)]) for f in (0.25, 0.5, 0.85, 0.9)}
        self.base = base

    def queries(self, nq, seed):
        g = torch.Generator(device=DEV).manual_seed(10_000 + seed)
        return self.mix.points(self.mix.labels(nq, g), g)


def _collection(c) -> _Collection:
    key = (c["dtype"], c["metric"], c["n"], c["d"], c["R"])
    if key not in _indices:
        _indices[key] = _Collection(*key)
        while len(_indices) > _HELD:
            _indices.popitem(last=False)
        torch.cuda.empty_cache()
    _indices.move_to_end(key)
    return _indices[key]


def _params(c, r):
    if "mode" not in c:
        return None
    more = {}
    if c.get("max_beam"):
        more["max_beam"] = c["max_beam"]
    if c.get("most"):
        more["max_results_per_query"] = c["most"]
    return rr.search_params(mode=c["mode"], beam=c["beam"], es_enable=c.get("es", False),
                            es_visit_limit=c.get("vl", 20), es_radius=c.get("esr", 1.0) * r,
                            precision=PRECISION[c.get("precision", "exact")],
                            result_capacity=c.get("cap", 0), cache_slots=c.get("cache_slots", 0),
                            waves_per_group=c.get("waves", 0), **more)


def prepare(case, seed):
    col = _collection(case)
    r = col.radii[case["nonempty"]]
    q = col.queries(case["nq"], seed)
    s = dict(case=case, index=col.index, q=q, r=r, params=_params(case, r))
    if case.get("radii"):
        g = torch.Generator(device=DEV).manual_seed(seed)
        s["r"] = r + abs(r) * 0.1 * (torch.rand(case["nq"], generator=g, device=DEV, dtype=torch.float64) - 0.5)
    if case["op"] == "serve":
        s["q"] = q.cpu().numpy()
        s["server"] = rr.Server(col.index, s["params"], slots=case["slots"], result_capacity=case["cap"])
        s["ids"], s["dists"] = np.zeros(_room(case), np.int32), np.zeros(_room(case), np.float32)
    elif case["op"] in ("search", "scan"):
        s["ids"] = torch.zeros(_room(case), dtype=torch.int32, device=DEV)
        s["dists"] = torch.zeros(_room(case), dtype=torch.float32 if case["dtype"] == "f32" else torch.int32,
                                 device=DEV)
    return s


def _room(c):
    """Entries of the output buffers: lists of any draw of the case fit."""
    return c.get("cap") or (1 << 21 if c["op"] == "scan" else c["nq"] * c.get("beam", 1))


def _keep(s, ids, dists, **more):
    """A program's own output buffers, of one size for every call; the entries
    past the lists stay zero."""
    n = min(len(ids), len(s["ids"]))
    s["ids"][:n] = ids[:n]
    s["dists"][:n] = dists[:n]
    return dict(ids=s["ids"], dists=s["dists"], **more)


def run(s):
    c, op = s["case"], s["case"]["op"]
    if op == "search":
        res = rr.range_search(s["index"], s["q"], s["r"], s["params"], with_stats=c.get("stats", False))
        more = {} if res.stats is None else {k: np.ascontiguousarray(res.stats[k]) for k in
                                             ("visits", "greedy_visits", "greedy_evals", "count")}
        return _keep(s, res.ids, res.dists, offsets=res.offsets, **more)
    if op == "scan":
        res = rr.brute_force(s["index"], s["q"], s["r"])
        return _keep(s, res.ids, res.dists, offsets=res.offsets)
    if op == "nn":
        return rr.nn_dist(s["index"], s["q"])
    if op == "radius":
        return rr.select_radius(s["index"], s["q"], [c["p"], c["p"] / 10])
    server, q = s["server"], s["q"]
    for tag in range(len(q)):
        server.submit(q[tag], s["r"], tag)
    server.drain(30.0)
    server.poll()
    got = [server.result(tag) for tag in range(len(q))]
    return _keep(s, np.concatenate([i for i, _ in got]), np.concatenate([d for _, d in got]),
                 counts=np.array([len(i) for i, _ in got]))


def work(case):
    """Dense scans: every row once, every product.  Searches: the adjacency
    rows of the points a beam of this width visits (the beam's own and a short
    way to them), a row for each neighbour seen for the first time (about
    half of them), and a visit for each result that the expansion adds."""
    c, es = case, ES[case["dtype"]]
    nq, n, d, R = c["nq"], c["n"], c["d"], c["R"]
    if c["op"] in ("scan", "nn", "radius"):
        return {"bytes": (n + nq) * d * es + nq * 8, "flops": 2.0 * n * nq * d}
    wide = c["beam"] if c["mode"] in ("plain", "es") else max(c["beam"], 8)
    visits = nq * (wide + 6.0)
    if c["mode"] == "doubling":
        visits = nq * 200.0
    elif c["mode"] == "adaptive":
        visits += nq * 40.0
    row = d * {"exact": es, "bf16": 2, "sq8": 1}[c.get("precision", "exact")]
    evals = visits * R * 0.5
    return {"bytes": visits * R * 4 + evals * row + nq * d * es, "flops": 2.0 * evals * d}


def exact(case, seed):
    """Dense scans in 64 bits from differences (or products); the lists of a
    graph search depend on the walk and have no such value."""
    if case["op"] not in ("scan", "nn", "radius"):
        return None
    col = _collection(case)
    q = col.queries(case["nq"], seed)
    if case["op"] == "nn" and case["dtype"] != "f32":
        return _pair_min(col.base, q, col.ip)
    x = col.base.double()
    q = q.double()
    r = col.radii[case["nonempty"]]
    lists, near, every = [], [], []
    for i in range(len(q)):
        dd = -(x * q[i]).sum(1) if col.ip else (x - q[i]).square().sum(1)
        if case["op"] == "nn":
            near.append(dd.min())
        elif case["op"] == "radius":
            every.append(dd)
        else:
            lists.append(dd[dd <= r].sort()[0])
    if case["op"] == "nn":
        return torch.stack(near)
    if case["op"] == "radius":
        every = torch.cat(every).sort()[0]
        k = [max(1, math.ceil(p * len(every))) for p in (case["p"], case["p"] / 10)]
        return np.array([float(every[j - 1]) for j in k])
    if case["dtype"] != "f32":
        return None
    out = torch.zeros(_room(case), dtype=torch.float64, device=DEV)
    lists = torch.cat(lists)[:len(out)]
    out[:len(lists)] = lists
    return dict(offsets=None, ids=None, dists=out)
