"""Searches of thousands of queries on the default schedule, which scan every query's nearest list first and the
others with its threshold.  Distances and labels equal those of the FP32 scan on a schedule set by hand, bit for bit."""
import numpy as np
import pytest

import paper_2601_11808_amd as sivf
from tests.invariants import check_dump

pytestmark = pytest.mark.gpu


# k up to 64 takes two phases from 8,000 queries and 4 probes on, k above 64 from 4,000; 3 probes and 7,999 and 3,999
# queries take one.  Lists shorter than k, empty ones, and a query's nearest list among them.
@pytest.mark.parametrize("metric,d", [(0, 24), (1, 24), (0, 100)])
def test_nearest_list_first(metric, d):
    rng = np.random.default_rng([31, metric, d])
    sizes = [6000, 2500, 700, 65, 64, 63, 9, 1, 0, 0] + list(rng.integers(0, 400, 50))
    nlist, n = len(sizes), sum(sizes)
    cent = (rng.standard_normal((nlist, d)) * 3).astype(np.float32)
    x = (cent[np.repeat(np.arange(nlist), sizes)] + rng.standard_normal((n, d))).astype(np.float32)
    x[1::53] = x[0::53][:x[1::53].shape[0]]          # equal rows under other ids
    ix = sivf.Index(d, nlist, cent, metric=metric, slab_capacity=32, num_slabs=n // 32 + 4 * nlist, id_capacity=n,
                    max_batch=n, max_queries=9000, max_k=128, max_nprobe=nlist)
    ix.add(x, rng.permutation(n))
    assert ix.sync() == 0
    q = (cent[rng.integers(0, nlist, 9000)] + rng.standard_normal((9000, d))).astype(np.float32)
    cases = [(9000, 10, 4), (8000, 1, 9), (8000, 64, 60), (8007, 33, 20), (7999, 10, 20), (8000, 10, 3), (4000, 65, 60),
             (4001, 128, 7), (3999, 100, 20)]
    got = [[t.cpu().numpy() for t in ix.search(q[:nq], k, p)] for nq, k, p in cases]
    assert ix.sync() == 0
    ix.set_search_schedule(8, 12, 0)
    for (nq, k, p), g in zip(cases, got):
        want = [t.cpu().numpy() for t in ix.search(q[:nq], k, p)]
        assert ix.sync() == 0
        assert all(np.array_equal(a.view(np.uint32), b.view(np.uint32)) for a, b in zip(g, want)), (nq, k, p)


def test_nearest_list_first_with_host_tier():
    """Lists moved to host memory: their results join the first phase's, and the second's."""
    rng = np.random.default_rng(32)
    d, nlist, n = 32, 20, 12000
    cent = (rng.standard_normal((nlist, d)) * 3).astype(np.float32)
    x = (cent[rng.integers(0, nlist, n)] + rng.standard_normal((n, d))).astype(np.float32)
    ix = sivf.Index(d, nlist, cent, slab_capacity=32, num_slabs=n // 32 + 4 * nlist, id_capacity=n, max_batch=n,
                    max_queries=8000, max_k=100, max_nprobe=nlist, delete_mode=sivf.DELETE_LAZY)
    ix.add(x, np.arange(n))
    q = (cent[rng.integers(0, nlist, 8000)] + rng.standard_normal((8000, d))).astype(np.float32)
    want = [[t.cpu().numpy() for t in ix.search(q, k, 8)] for k in (10, 100)]
    ix.tier_attach(n // 32 + 4 * nlist)
    ix.tier_offload([0, 3, 4, 11])
    assert ix.sync() == 0
    for k, w in zip((10, 100), want):
        got = [t.cpu().numpy() for t in ix.search(q, k, 8)]
        assert ix.sync() == 0
        assert all(np.array_equal(a.view(np.uint32), b.view(np.uint32)) for a, b in zip(got, w)), k


# per-list counts by blocks of 4,096 entries from 65,536 on: either side of the line, a ragged last block, and upserts,
# repeated and absent ids within such a batch; lazy deletes count through the same blocks
@pytest.mark.parametrize("lazy", [False, True])
@pytest.mark.parametrize("n", [65535, 65536, 69633])
def test_mutation_counts_of_large_batches(n, lazy):
    rng = np.random.default_rng([33, n])
    d, nlist, cap = 4, 77, 2 * n
    cent = (rng.standard_normal((nlist, d)) * 9).astype(np.float32)
    share = rng.random(nlist) ** 4
    x = (cent[rng.choice(nlist, n, p=share / share.sum())] + rng.standard_normal((n, d))).astype(np.float32)
    slabs = 2 * n // 32 + 4 * nlist
    ix = sivf.Index(d, nlist, cent, slab_capacity=32, num_slabs=slabs, id_capacity=cap, max_batch=n, max_queries=16,
                    max_k=16, max_nprobe=16, delete_mode=sivf.DELETE_LAZY if lazy else sivf.DELETE_COMPACT)
    where = {}

    def add(rows, ids):
        ix.add(rows, ids)
        assert ix.sync() == 0
        for i, u in enumerate(ids):
            where[int(u)] = rows[i]

    def check():
        got = ix.membership()
        assert sum(len(v) for v in got.values()) == len(where)
        check_dump(ix.dump(), 32, slabs, lazy=lazy)
        live = np.fromiter(where, np.int64)
        np.testing.assert_array_equal(ix.get_rows(live).cpu().numpy(), np.stack(list(where.values())))

    add(x, rng.permutation(cap)[:n])
    check()
    ids = rng.permutation(cap)[:n]
    ids[5::7] = ids[0::7][:ids[5::7].shape[0]]       # the last of equal ids wins
    add(x[::-1].copy(), ids)
    check()
    gone = rng.permutation(cap)[:n]                  # some of them hold nothing
    removed = ix.remove(gone)
    assert ix.sync() == 0
    assert int(removed.item()) == sum(where.pop(int(u), None) is not None for u in gone)
    check()


def test_nearest_list_first_in_a_graph():
    """A captured step of a two-phase search and a delete counted by large blocks: every replay equals the eager
    step on a second index."""
    import torch

    rng = np.random.default_rng(34)
    d, nlist, b, nq = 16, 40, 65536, 8000
    cent = (rng.standard_normal((nlist, d)) * 4).astype(np.float32)
    ring = (cent[rng.integers(0, nlist, 4 * b)] + rng.standard_normal((4 * b, d))).astype(np.float32)

    def index():
        ix = sivf.Index(d, nlist, cent, slab_capacity=64, num_slabs=4 * b // 64 + 4 * nlist, id_capacity=4 * b, max_batch=b,
                        max_queries=nq, max_k=32, max_nprobe=8)
        ix.add(ring[:b], np.arange(b))
        assert ix.sync() == 0
        return ix

    eager, ix = index(), index()
    dev = dict(device="cuda:0")
    x, q = torch.zeros(b, d, **dev), torch.zeros(nq, d, **dev)
    ids, rm = torch.zeros(b, dtype=torch.int64, **dev), torch.zeros(b, dtype=torch.int64, **dev)
    dist, lab = torch.empty(nq, 20, **dev), torch.empty(nq, 20, dtype=torch.int64, **dev)
    nrem = torch.zeros(1, dtype=torch.int64, **dev)
    g = ix.step_graph(x, ids, q, 20, 8, rm, dist, lab, nrem)
    for t in range(1, 4):
        new = np.arange(t * b, (t + 1) * b)
        qt = (cent[rng.integers(0, nlist, nq)] + rng.standard_normal((nq, d))).astype(np.float32)
        x.copy_(torch.from_numpy(ring[new]))
        ids.copy_(torch.from_numpy(new))
        rm.copy_(torch.from_numpy(new - b))
        q.copy_(torch.from_numpy(qt))
        g.launch()
        assert ix.sync() == 0
        wd, wl, wn = eager.step(ring[new], new, qt, 20, 8, new - b)
        assert eager.sync() == 0
        assert torch.equal(dist.view(torch.int32), wd.view(torch.int32)) and torch.equal(lab, wl)
        assert int(nrem.item()) == int(wn.item()) == b
        ix.search(qt[:5], 3, 2)                      # eager work between the replays
        assert {l: sorted(v) for l, v in ix.membership().items()} == {l: sorted(v) for l, v in eager.membership().items()}
    g.close()
