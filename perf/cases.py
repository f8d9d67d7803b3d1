"""Performance cases of the streaming IVF index: what a program that keeps a
GPU-resident window of vectors has it do, through the public entry points.

Every case is one pass of one of these operations, on an index that has been
filled beforehand with `n` vectors of dimension `d`:

  search    Index.search of `nq` queries (with `uneven`, per-query k out of
            {1, 10, 100} and per-query nprobe, as a mixed batch has)
  step      Index.step: insert `batch` vectors, search `nq` queries, delete
            `batch` ids (the oldest, or with `scatter` ids spread over the
            whole window); with `graph` the step is a captured HIP graph and
            its input buffers are refilled before each launch
  lazy      the same step on an index with lazy deletes, followed by
            Index.compact, as a window of constant size needs it
  registry  Registry.add, .search and .remove with external 64-bit ids
  server    a burst of requests through Server: searches of mixed sizes
            around two inserts and a delete, then a wait for every ticket

A window slides over a ring of n + batch vectors: each pass inserts the block
of the ring that is out of the window and deletes the next one, so the window
keeps its size and a pass can be repeated without end.  Schedules are the
library's defaults.

Inputs follow the workloads of this repository: `int` data are whole values
0..255 around cluster means (d <= 128) with centroids from a few Lloyd
iterations, so list lengths are uneven as k-means leaves them; `real` data are
the unrounded mixture with the means as centroids, with `skew` under Zipf(1.1)
cluster weights; `unit` data are normalised for inner-product search.
"""
import math

import torch

import paper_2601_11808_amd as sivf

DEV = "cuda:0"
K_CHOICES = (1, 10, 100)


def listed():
    f = dict(metric="l2", dtype="f32", data="int", d=128, slab=64, k=10)
    return [
        # an interactive lookup: one query against a 1M window, where latency is everything
        dict(f, name="one_query", op="search", n=1_000_000, nlist=1024, nq=1, nprobe=32),
        # a small ragged batch: inner product, d no multiple of 8, odd counts, short slabs
        dict(f, name="few_queries_ip", op="search", n=300_001, nlist=1000, nq=37, nprobe=16, d=100, metric="ip",
             data="unit", slab=32, k=7),
        # the sliding window at its usual size: +10k / 10k queries / -10k on 1M vectors
        dict(f, name="window_step", op="step", n=1_000_000, nlist=1024, nq=10_000, nprobe=32, batch=10_000),
        # the latency-bound window: small updates and few queries on 200k vectors
        dict(f, name="small_step", op="step", n=200_000, nlist=1024, nq=100, nprobe=16, batch=1000),
        # wide rows (global image descriptors): +5k / -5k on 100k vectors of 960 values
        dict(f, name="wide_step", op="step", n=100_000, nlist=512, nq=1000, nprobe=16, batch=5000, d=960,
             data="real"),
        # a mixed batch: skewed list lengths, every query with its own k and nprobe
        dict(f, name="uneven_batch", op="search", n=5_000_000, nlist=2048, nq=32_000, nprobe=128, data="real", skew=True,
             uneven=True, k=100),
        # reduced precision: bf16 slabs and exact re-rank, inner product over 10M unit vectors
        dict(f, name="bf16_search", op="search", n=10_000_000, nlist=4096, nq=16_000, nprobe=64, d=96, metric="ip",
             dtype="bf16", data="unit", slab=128),
        # one search of a serving process: a few hundred queries over many lists, fp16 slabs
        dict(f, name="fp16_many_lists", op="search", n=8_000_000, nlist=16_384, nq=477, nprobe=40, dtype="f16",
             data="real", slab=128),
        # the serving loop itself: queued searches of mixed sizes around inserts and a delete
        dict(f, name="server_burst", op="server", n=2_000_000, nlist=4096, nq=600, nprobe=32, batch=20_000,
             dtype="f16", data="real", slab=128, requests=12),
        # bulk turnover: a quarter of the window replaced, the deleted ids spread over all slabs
        dict(f, name="bulk_turnover", op="step", n=1_000_000, nlist=1024, nq=64, nprobe=8, batch=250_000,
             scatter=True),
        # lazy deletes with the compaction that a steady window needs
        dict(f, name="lazy_step", op="lazy", n=500_000, nlist=1024, nq=1000, nprobe=16, batch=10_000),
        # external ids: a small registry window
        dict(f, name="registry_step", op="registry", n=200_000, nlist=512, nq=200, nprobe=16, batch=2000),
    ]


def _between(rng, lo, hi):
    """A whole number in [lo, hi], spread over its logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    op = rng.choice(["search", "search", "search", "step", "step", "uneven", "reduced", "reduced", "lazy", "registry",
                     "server"])
    c = dict(op="search" if op in ("uneven", "reduced") else op, metric="l2", dtype="f32", data="int",
             slab=rng.choice([32, 64, 128]), k=_between(rng, 1, 64))
    if op == "uneven":
        c.update(n=_between(rng, 200_000, 5_000_000), d=rng.choice([96, 100, 128]), nlist=_between(rng, 1024, 2048),
                 nq=_between(rng, 100, 32_000), nprobe=_between(rng, 16, 128), data="real", skew=True, uneven=True,
                 k=100)
    elif op in ("reduced", "server"):
        c.update(dtype=rng.choice(["bf16", "f16"]), slab=rng.choice([64, 128]), k=_between(rng, 1, 16),
                 data="real", d=rng.choice([64, 96, 100, 128]), nprobe=_between(rng, 8, 64))
        if rng.random() < 0.4:
            c.update(metric="ip", data="unit")
        if op == "server":
            c.update(n=_between(rng, 200_000, 2_000_000), nlist=_between(rng, 512, 4096), nq=_between(rng, 8, 600),
                     batch=_between(rng, 500, 20_000), requests=rng.randint(4, 12))
        else:
            c.update(n=_between(rng, 200_000, 8_000_000), nlist=_between(rng, 512, 8192), nq=_between(rng, 1, 16_000))
    else:
        c.update(n=_between(rng, 50_000, 1_000_000), nlist=_between(rng, 100, 2048), nq=_between(rng, 1, 10_000),
                 nprobe=_between(rng, 1, 64), d=rng.choice([32, 64, 96, 100, 127, 128]))
        shape = rng.random()
        if shape < 0.2:      # wide rows
            c.update(d=rng.choice([200, 256, 384, 768, 960]), data="real", n=_between(rng, 20_000, 100_000),
                     nlist=_between(rng, 64, 512), nq=_between(rng, 1, 1000), nprobe=_between(rng, 1, 16))
        elif shape < 0.45:   # inner product on unit vectors
            c.update(metric="ip", data="unit")
        if op != "search":
            c["batch"] = _between(rng, 100, max(200, c["n"] // 10))
        if op == "step":
            c["scatter"] = rng.random() < 0.4
            c["graph"] = rng.random() < 0.25
        if op == "registry":
            c.update(nq=min(c["nq"], 2000), batch=min(c["batch"], 20_000))
    c["nprobe"] = min(c["nprobe"], c["nlist"])
    return c


# ---- inputs --------------------------------------------------------------

def _gen(seed, tag):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed * 1_000_003 + tag)
    return g


def _mixture(case, seed):
    """Means and weights of the clusters (as many as lists)."""
    g = _gen(seed, 1)
    m = torch.rand((case["nlist"], case["d"]), generator=g, device=DEV) * 255.0
    if case["data"] == "unit":
        m = torch.nn.functional.normalize(torch.randn(m.shape, generator=g, device=DEV), dim=1)
    w = None
    if case.get("skew"):
        r = torch.randperm(case["nlist"], generator=g, device=DEV).double() + 1.0
        w = r ** -1.1
    return m, w


def _sample(case, seed, tag, means, weights, n):
    g = _gen(seed, tag)
    if weights is None:
        comp = torch.randint(0, means.shape[0], (n,), generator=g, device=DEV)
    else:   # inverse transform: deterministic, and no limit on n
        cdf = torch.cumsum(weights / weights.sum(), 0)
        u = torch.rand(n, generator=g, device=DEV, dtype=torch.float64)
        comp = torch.searchsorted(cdf, u).clamp_(max=means.shape[0] - 1)
    x = torch.randn((n, case["d"]), generator=g, device=DEV)
    if case["data"] == "unit":
        x.div_(math.sqrt(50.0)).add_(means[comp])
        return torch.nn.functional.normalize(x, dim=1)
    x.mul_(48.0).add_(means[comp])
    return x.round_().clamp_(0, 255) if case["data"] == "int" else x


def _lloyd(sample, nlist, iters=4):
    """Lloyd iterations whose every sum is a whole number below 2^24 (values
    0..255, d <= 128, at most 65,536 rows, rounded centroids), so the result
    does not depend on any order of summation."""
    c = sample[:nlist].clone()
    for _ in range(iters):
        score = (c * c).sum(1)[None, :] - 2.0 * (sample @ c.t())
        a = score.argmin(1)
        s = torch.zeros_like(c).index_add_(0, a, sample)
        cnt = torch.bincount(a, minlength=nlist).to(c.dtype)
        c = torch.where(cnt[:, None] > 0, torch.round(s / cnt.clamp(min=1)[:, None]), c)
    return c


def _ring(case):
    """(vectors of the ring, passes until it repeats): the window's vectors
    and one block more, in whole blocks."""
    b = case.get("batch", 0)
    if not b:
        return case["n"], 1
    blocks = max(2, round(case["n"] / b)) + 1
    return blocks * b, blocks


def _inputs(case, seed):
    """Everything random of a case: ring vectors, their ids, centroids and
    queries."""
    means, weights = _mixture(case, seed)
    total, _ = _ring(case)
    if case["data"] == "int":
        cent = _lloyd(_sample(case, seed, 2, means, weights, 65_536), case["nlist"])
    else:
        cent = means
    x = _sample(case, seed, 3, means, weights, total)
    q = _sample(case, seed, 4, means, weights, case["nq"])
    ids = torch.arange(total, device=DEV)
    if case["op"] == "registry":   # sparse keys: an odd multiplier permutes the 63-bit range
        ids = (ids * 0x2545F4914F6CDD1D) & 0x7FFFFFFFFFFFFFFF
    kpq = npq = None
    if case.get("uneven"):
        g = _gen(seed, 5)
        kpq = torch.tensor(K_CHOICES, dtype=torch.int32, device=DEV)[
            torch.randint(0, 3, (case["nq"],), generator=g, device=DEV)]
        npq = torch.randint(max(1, case["nprobe"] // 16), case["nprobe"] + 1, (case["nq"],), generator=g, device=DEV,
                            dtype=torch.int32)
    return x, ids, cent, q, kpq, npq


def _blocks(case, t):
    """(block inserted, block deleted) by pass t."""
    _, blocks = _ring(case)
    return (blocks - 1 + t) % blocks, t % blocks


def _base_order(case, seed, total):
    """Row order in which the window is filled.  With `scatter` the rows of a
    block are spread over the whole fill, so deleting a block touches every
    slab; otherwise blocks follow each other, oldest first."""
    n = total - case.get("batch", 0)
    if case.get("scatter"):
        return torch.randperm(n, generator=_gen(seed, 6), device=DEV)
    return None


def _request_sizes(case):
    """Queries of each search of a server burst: about geometric steps from 1
    to nq, small and large mixed."""
    r = case["requests"]
    sizes = [max(1, int(round(case["nq"] ** (i / max(1, r - 1))))) for i in range(r)]
    return [sizes[(i * 5) % r] if math.gcd(5, r) == 1 else sizes[i] for i in range(r)]


def prepare(case, seed):
    x, ids, cent, q, kpq, npq = _inputs(case, seed)
    total, _ = _ring(case)
    b = case.get("batch", 0)
    load = min(total, 1 << 20)
    C = case["slab"]
    reduced = case["dtype"] != "f32"
    lazy = case["op"] == "lazy"
    burst = sum(_request_sizes(case)) if case["op"] == "server" else 0
    ix = sivf.Index(
        case["d"], case["nlist"], cent, metric=sivf.IP if case["metric"] == "ip" else sivf.L2, slab_capacity=C,
        num_slabs=int(1.15 * (case["n"] + 3 * b) / C) + 2 * case["nlist"] + (total // (2 * C) if lazy else 0),
        id_capacity=total, max_batch=max(load, b), max_queries=max(1024, case["nq"], 2 * burst),
        max_k=max(16, case["k"]), max_nprobe=max(64, case["nprobe"]),
        storage={"f32": sivf.F32, "bf16": sivf.BF16, "f16": sivf.F16}[case["dtype"]], rerank_factor=4 if reduced else 0,
        delete_mode=sivf.DELETE_LAZY if lazy else sivf.DELETE_COMPACT, device=DEV)
    s = dict(case=case, ix=ix, x=x, ids=ids, q=q, kpq=kpq, npq=npq, t=0, blocks=[])
    into = ix
    if case["op"] == "registry":
        into = s["reg"] = sivf.Registry(ix)
    order = _base_order(case, seed, total)
    n = total - b
    for i in range(0, n, load):
        rows = slice(i, min(i + load, n)) if order is None else order[i:i + load]
        into.add(x[rows], ids[rows])
    ix.check()
    if b:   # the blocks of the ring, as a program that receives them has them
        s["blocks"] = [(x[i:i + b], ids[i:i + b]) for i in range(0, total, b)]
    if case.get("graph"):
        k, nq = case["k"], case["nq"]
        s["buf"] = [torch.empty_like(s["blocks"][0][0]), torch.empty_like(s["blocks"][0][1]),
                    torch.empty_like(s["blocks"][0][1])]
        s["dist"] = torch.empty((nq, k), device=DEV)
        s["lab"] = torch.empty((nq, k), dtype=torch.int64, device=DEV)
        s["nrem"] = torch.zeros(1, dtype=torch.int64, device=DEV)
        s["graph"] = ix.step_graph(s["buf"][0], s["buf"][1], q, k, case["nprobe"], s["buf"][2], s["dist"], s["lab"],
                                   s["nrem"])
    if case["op"] == "server":
        s["server"] = sivf.Server(ix)
        s["qs"] = [q[:m].contiguous() for m in _request_sizes(case)]
        h = b // 2 or 1
        s["halves"] = [((xb[:h], ib[:h]), (xb[h:], ib[h:])) for xb, ib in s["blocks"]]
    return s


# ---- one pass ------------------------------------------------------------

def run(s):
    c, ix = s["case"], s["ix"]
    k, nprobe = c["k"], c["nprobe"]
    if c["op"] == "search":
        dist, lab = ix.search(s["q"], k, nprobe, k_per_query=s["kpq"], nprobe_per_query=s["npq"])
        return {"dist": dist, "labels": lab}
    new, old = _blocks(c, s["t"])
    s["t"] += 1
    (xb, ib), (_, ob) = s["blocks"][new], s["blocks"][old]
    if c.get("graph"):
        for dst, src in zip(s["buf"], (xb, ib, ob)):
            dst.copy_(src)
        s["graph"].launch()
        return {"dist": s["dist"], "labels": s["lab"], "removed": s["nrem"]}
    if c["op"] == "registry":
        reg = s["reg"]
        reg.add(xb, ib)
        dist, lab = reg.search(s["q"], k, nprobe)
        return {"dist": dist, "labels": lab, "removed": reg.remove(ob)}
    if c["op"] == "server":
        return _burst(s, new, old)
    dist, lab, nrem = ix.step(xb, ib, s["q"], k, nprobe, ob)
    if c["op"] == "lazy":
        return {"dist": dist, "labels": lab, "removed": nrem, "compacted": ix.compact(0.1)}
    return {"dist": dist, "labels": lab, "removed": nrem}


def _burst(s, new, old):
    """A third of the searches, an insert, another third, the delete and the
    second insert, then the rest; returns when every request is done."""
    c, srv, qs = s["case"], s["server"], s["qs"]
    (first, second), ob = s["halves"][new], s["blocks"][old][1]
    tickets, out = [], []
    cut = [len(qs) // 3, 2 * len(qs) // 3]
    removed = None
    for i, q in enumerate(qs):
        if i == cut[0]:
            tickets.append(srv.add(*first))
        if i == cut[1]:
            t, removed = srv.remove(ob)
            tickets += [t, srv.add(*second)]
        t, dist, lab = srv.search(q, c["k"], c["nprobe"])
        tickets.append(t)
        out.append((dist, lab))
    for t in tickets:
        srv.wait(t)
    return {"dist": [d for d, _ in out], "labels": [v for _, v in out], "removed": removed}


# ---- what a pass cannot do without -----------------------------------------

def work(case):
    d, nlist, n, k = case["d"], case["nlist"], case["n"], case["k"]
    nq = sum(_request_sizes(case)) if case["op"] == "server" else case["nq"]
    nprobe = case["nprobe"]
    if case.get("uneven"):
        nprobe = (max(1, nprobe // 16) + nprobe) / 2
    elem = 4 if case["dtype"] == "f32" else 2
    evals = nq * nprobe * n / nlist
    byts = nq * d * 4 + nlist * d * 4 + min(n, evals) * (elem * d + 4) + nq * k * 12
    flops = 2.0 * nq * nlist * d + 2.0 * evals * d
    b = case.get("batch", 0)
    if b:
        byts += b * (4 * d + 4 * d + 8 + 8) + (b * 2 * d if elem == 2 else 0) + b * 12
        flops += 2.0 * b * nlist * d
    return {"bytes": byts, "flops": flops}


# ---- the same in 64 bits ---------------------------------------------------

def _scores(a, b, metric):
    """Squared L2 distances, or negated inner products, of a's rows to b's."""
    s = a @ b.t()
    if metric == "ip":
        return -s
    return (a * a).sum(1)[:, None] + (b * b).sum(1)[None, :] - 2.0 * s


def _exact_search(case, rows, assign, cent, q, kpq, npq):
    """Distances of the k nearest of `rows` within each query's nprobe nearest
    lists; `assign` is each row's list."""
    m, k, nprobe = case["metric"], case["k"], case["nprobe"]
    inf = float("inf")
    q = q.double()
    probes = torch.cat([_scores(c, cent, m).topk(nprobe, dim=1, largest=False).indices
                        for c in q.split(4096)])
    use = torch.ones_like(probes, dtype=torch.bool)
    if npq is not None:
        use = torch.arange(nprobe, device=DEV)[None, :] < npq[:, None]
    order = torch.sort(assign, stable=True).indices
    ends = torch.cumsum(torch.bincount(assign, minlength=case["nlist"]), 0).tolist()
    qi, pi = torch.nonzero(use, as_tuple=True)
    by = torch.sort(probes[qi, pi], stable=True).indices
    pends = torch.cumsum(torch.bincount(probes[qi, pi], minlength=case["nlist"]), 0).tolist()
    best = torch.full((q.shape[0], nprobe, k), inf, dtype=torch.float64, device=DEV)
    a = pa = 0
    for e, pe in zip(ends, pends):
        if e > a and pe > pa:
            x = rows[order[a:e]].double()
            for lo in range(pa, pe, max(1, (1 << 27) // (e - a))):
                sel = by[lo:min(pe, lo + max(1, (1 << 27) // (e - a)))]
                sc = _scores(q[qi[sel]], x, m)
                kk = min(k, e - a)
                best[qi[sel], pi[sel], :kk] = sc.topk(kk, dim=1, largest=False).values
        a, pa = e, pe
    dist = best.reshape(q.shape[0], -1)
    dist = torch.cat([dist, torch.full((q.shape[0], k), inf, dtype=torch.float64, device=DEV)], 1)
    dist = dist.topk(k, dim=1, largest=False).values.sort(dim=1).values
    if kpq is not None:
        dist[torch.arange(k, device=DEV)[None, :] >= kpq[:, None]] = inf
    return -dist if m == "ip" else dist


def exact(case, seed):
    nq = sum(_request_sizes(case)) if case["op"] == "server" else case["nq"]
    evals = work(case)["flops"] / 2 / case["d"] - nq * case["nlist"]
    if (evals * (8 if case.get("skew") else 2.5) + case["n"] * case["nlist"]) * 2 * case["d"] > 6e14:
        return None   # more than some 20 seconds of fp64 products
    x, _, cent, q, kpq, npq = _inputs(case, seed)
    total, blocks = _ring(case)
    cent = cent.double()
    assign = torch.cat([_scores(c.double(), cent, case["metric"]).argmin(1) for c in x.split(1 << 17 if
                        case["nlist"] <= 4096 else 1 << 15)])
    b = case.get("batch", 0)

    def search(live, q):
        if live is None:
            return _exact_search(case, x, assign, cent, q, kpq, npq)
        return _exact_search(case, x[live], assign[live], cent, q, kpq, npq)

    if case["op"] == "search":
        return {"dist": search(None, q), "labels": None}
    new, old = _blocks(case, 0)
    if case["op"] != "server":   # a step searches between its insert and its delete: the whole ring is live
        out = {"dist": search(None, q), "labels": None, "removed": None}
        return dict(out, compacted=None) if case["op"] == "lazy" else out
    sizes, h = _request_sizes(case), b // 2 or 1
    cut = [len(sizes) // 3, 2 * len(sizes) // 3]
    row = torch.arange(total, device=DEV)
    first = (row >= new * b) & (row < new * b + h)
    added, gone = (row >= new * b) & (row < (new + 1) * b), (row >= old * b) & (row < (old + 1) * b)
    dist = []
    for lo, hi, live in ((0, cut[0], ~added), (cut[0], cut[1], ~added | first), (cut[1], len(sizes), ~gone)):
        if hi > lo:
            d = search(live, torch.cat([q[:m] for m in sizes[lo:hi]]))
            dist += list(d.split(sizes[lo:hi]))
    return {"dist": dist, "labels": [None] * len(sizes), "removed": None}
