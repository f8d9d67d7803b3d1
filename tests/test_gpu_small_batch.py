"""Searches of few queries, on the default (batch-dependent) schedule: tiles of 2
and 4 queries, lists split into short chunks so that few (query, list) pairs
fill the chip, and the merge by one or four waves per query.  Results equal the
oracle's, and those of a schedule set by hand, bit for bit."""
import numpy as np
import pytest

import oracle
import paper_2601_11808_amd as sivf
from tests.gpu_common import compare_results
from tests.invariants import check_dump, same_membership

pytestmark = pytest.mark.gpu


def _index(seed, d, sizes, metric, C, max_queries, max_k, max_nprobe):
    rng = np.random.default_rng(seed)
    nlist = len(sizes)
    cent = (rng.standard_normal((nlist, d)) * 6).astype(np.float32)
    lab = np.repeat(np.arange(nlist), sizes)
    x = (cent[lab] + rng.standard_normal((lab.shape[0], d))).astype(np.float32)
    x[1::97] = x[0::97][:x[1::97].shape[0]]          # equal rows under other ids
    ids = np.arange(x.shape[0])
    rng.shuffle(x)
    slabs = x.shape[0] // C + 2 * nlist + 8
    ix = sivf.Index(d, nlist, cent, metric=metric, slab_capacity=C, num_slabs=slabs, id_capacity=x.shape[0],
                    max_batch=x.shape[0], max_queries=max_queries, max_k=max_k, max_nprobe=max_nprobe)
    ref = oracle.OracleIndex(d, nlist, cent, metric, C, slabs, x.shape[0])
    ix.add(x, ids)
    assert ix.sync() == 0 and ref.add(x, ids) == 0
    q = (cent[rng.integers(0, nlist, max_queries)] + rng.standard_normal((max_queries, d))).astype(np.float32)
    q[0] = x[5]
    return ix, ref, q


# d: float4 rows read through the scalar cache, and rows staged in LDS (d % 4 != 0)
@pytest.mark.parametrize("metric,d,C", [(0, 32, 64), (1, 30, 32), (0, 300, 128)])
def test_few_queries_split_lists(metric, d, C):
    sizes = [30000, 9000, 2000, 700, 129, 128, 64, 1, 0] + [37] * 71
    ix, ref, q = _index([21, metric, d], d, sizes, metric, C, 1000, 128, 80)
    default = ix.search_schedule()[0]
    for nq, k, nprobe in [(1, 1, 1), (1, 10, 80), (1, 128, 80), (2, 65, 9), (5, 64, 3), (70, 16, 7), (768, 10, 2),
                          (769, 100, 1)]:
        gd, gl = ix.search(q[:nq], k, nprobe)
        assert ix.sync() == 0
        st, rd, rl = ref.search(q[:nq], k, nprobe)
        assert st == 0
        assert compare_results(gd.cpu().numpy(), gl.cpu().numpy(), rd, rl) == 0, (nq, k, nprobe)
    assert ix.search_schedule()[0] == default        # the rule changes no setting
    # the same batch under every schedule the caller can set
    kpq = np.random.default_rng(3).choice(np.array([0, 1, 10, 100, 128], np.int32), 40)
    npq = np.random.default_rng(4).integers(1, 81, 40).astype(np.int32)
    want = [t.cpu().numpy() for t in ix.search(q[:40], 128, 1, k_per_query=kpq, nprobe_per_query=npq)]
    st, rd, rl = ref.search(q[:40], 128, 1, k_per_query=kpq, nprobe_per_query=npq)
    assert st == 0 and compare_results(*want, rd, rl) == 0
    for sched in [(4, 6, 0), (4, 14, 1), (8, 9, 0)] + ([(16, 6, 0), (16, 13, 1)] if d <= 256 else []):
        ix.set_search_schedule(*sched)
        got = [t.cpu().numpy() for t in ix.search(q[:40], 128, 1, k_per_query=kpq, nprobe_per_query=npq)]
        assert all(np.array_equal(a.view(np.uint32), b.view(np.uint32)) for a, b in zip(want, got)), sched


def test_few_queries_small_buffers():
    """An index planned for one query of eight probes: the split stays within its buffers."""
    sizes = [20000, 5000, 300] + [5] * 13
    ix, ref, q = _index([22], 16, sizes, 0, 64, 1, 128, 8)
    for k in (1, 128):
        gd, gl = ix.search(q[:1], k, 8)
        assert ix.sync() == 0
        st, rd, rl = ref.search(q[:1], k, 8)
        assert st == 0 and compare_results(gd.cpu().numpy(), gl.cpu().numpy(), rd, rl) == 0


# the selection kernels' edges: lists per thread (1,024 / 2,048 / 4,096 / 16,384 and past them), rows per launch
# (the wave kernel from 1,536 rows), probes 64 / 65 / 128 / 129, and the untiled GEMM's ragged last lists
@pytest.mark.parametrize("nlist,nq,nprobe", [(17, 3, 17), (1024, 5, 64), (1023, 1536, 64), (1025, 1536, 65),
                                             (2048, 1540, 128), (2048, 1536, 129), (2049, 40, 33), (4097, 7, 128),
                                             (16384, 3, 64), (16400, 3, 200)])
@pytest.mark.parametrize("metric", [0, 1])
def test_probe_selection_edges(nlist, nq, nprobe, metric):
    """Probes in order, and a search over the unordered set, equal the oracle's; centroids repeat (exact ties)
    and a query equals one."""
    rng = np.random.default_rng([23, nlist, nprobe, metric])
    d = 24
    cent = rng.integers(-4, 5, (nlist, d)).astype(np.float32)
    cent[nlist // 2] = cent[0]
    q = rng.integers(-4, 5, (nq, d)).astype(np.float32)
    q[0] = cent[0]
    x = rng.integers(-4, 5, (4000, d)).astype(np.float32)
    slabs = 4000 // 4 + nlist + 8
    ix = sivf.Index(d, nlist, cent, metric=metric, slab_capacity=4, num_slabs=slabs, id_capacity=4000, max_batch=4000,
                    max_queries=2000, max_k=16, max_nprobe=200)
    ref = oracle.OracleIndex(d, nlist, cent, metric, 4, slabs, 4000)
    ix.add(x, np.arange(4000))
    assert ix.sync() == 0 and ref.add(x, np.arange(4000)) == 0
    np.testing.assert_array_equal(ix.probe(q, nprobe).cpu().numpy(), oracle.probe(q, cent, nprobe, metric))
    gd, gl = ix.search(q, 7, nprobe)
    assert ix.sync() == 0
    st, rd, rl = ref.search(q, 7, nprobe)
    assert st == 0 and compare_results(gd.cpu().numpy(), gl.cpu().numpy(), rd, rl) == 0


# the move of survivors: groups of 8 chunks (d past 32 and 64), runs of lists shorter and longer than a wave, and a
# whole list
@pytest.mark.parametrize("d,C,storage", [(5, 4, 0), (33, 64, 0), (72, 32, 1), (260, 16, 0)])
def test_delete_moves(d, C, storage):
    rng = np.random.default_rng([24, d])
    sizes = [700, 1, 2, 3, 300, 0] + [5] * 90
    nlist, n = len(sizes), sum(sizes)
    cent = (rng.standard_normal((nlist, d)) * 8).astype(np.float32)
    x = (cent[np.repeat(np.arange(nlist), sizes)] + rng.standard_normal((n, d))).astype(np.float32)
    ids = rng.permutation(n)
    slabs = n // C + 2 * nlist
    ix = sivf.Index(d, nlist, cent, slab_capacity=C, num_slabs=slabs, id_capacity=n, max_batch=n, max_queries=16,
                    max_k=16, max_nprobe=16, storage=storage, rerank_factor=4 if storage else 0)
    ref = oracle.OracleIndex(d, nlist, cent, 0, C, slabs, n)
    ix.add(x, ids)
    assert ix.sync() == 0 and ref.add(x, ids) == 0
    row_of = np.argsort(ids)
    for share in (0.02, 0.3, 0.5, 1.0):
        live = ref.live_ids() if hasattr(ref, "live_ids") else np.concatenate(list(ref.membership().values()))
        rm = rng.choice(live, max(1, int(share * live.shape[0])), replace=False).astype(np.int64)
        nr = ix.remove(rm)
        assert ix.sync() == 0 and int(nr.item()) == rm.shape[0]
        assert ref.remove(rm)[0] == 0
        gm, om = ix.membership(), ref.membership()
        assert gm.keys() == om.keys() and all(np.array_equal(gm[l], np.sort(om[l])) for l in om)
        keep = np.setdiff1d(live, rm)
        if keep.shape[0]:
            np.testing.assert_array_equal(ix.get_rows(keep).cpu().numpy(), x[row_of[keep]])


# compaction takes the holes by validity words: slabs shorter than a word, of one, and of two
@pytest.mark.parametrize("C", [4, 32, 64, 128])
def test_compaction_slab_words(C):
    rng = np.random.default_rng([25, C])
    d, sizes = 20, [1500, 1, 2, 300, 0, 64, 65, 257] + [90] * 20
    nlist, n = len(sizes), sum(sizes)
    cent = (rng.standard_normal((nlist, d)) * 8).astype(np.float32)
    x = (cent[np.repeat(np.arange(nlist), sizes)] + rng.standard_normal((n, d))).astype(np.float32)
    ids = rng.permutation(n)
    slabs = n // C + 2 * nlist
    ix = sivf.Index(d, nlist, cent, slab_capacity=C, num_slabs=slabs, id_capacity=n, max_batch=n, max_queries=64,
                    max_k=16, max_nprobe=16, delete_mode=sivf.DELETE_LAZY)
    ref = oracle.OracleIndex(d, nlist, cent, 0, C, slabs, n)
    ix.add(x, ids)
    assert ix.sync() == 0 and ref.add(x, ids) == 0
    q = x[rng.integers(0, n, 64)]
    live = ids.copy()
    for share in (0.01, 0.3, 0.6, 1.0):
        rm = rng.choice(live, max(1, int(share * live.shape[0])), replace=False).astype(np.int64)
        ix.remove(rm)
        dead = int(ix.compact(0.0).item())
        assert ix.sync() == 0 and ref.remove(rm)[0] == 0 and dead == rm.shape[0]
        live = np.setdiff1d(live, rm)
        check_dump(ix.dump(), C, slabs, lazy=True)
        assert same_membership(ix.membership(), ref.membership())
        gd, gl = ix.search(q, 10, 16)
        assert ix.sync() == 0
        st, rd, rl = ref.search(q, 10, 16)
        assert st == 0 and compare_results(gd.cpu().numpy(), gl.cpu().numpy(), rd, rl) == 0


# rows staged in pieces of 64 chunks of 4 values: one whole piece, one and a remainder, several, a last wave of fewer
# entries than it holds, and either side of the batch from which wide rows are not staged
@pytest.mark.parametrize("d,n", [(256, 16), (260, 17), (512, 33), (1028, 47), (260, 8192), (260, 8193)])
def test_insert_wide_rows(d, n):
    rng = np.random.default_rng([26, d])
    cent = rng.standard_normal((5, d)).astype(np.float32)
    x = (cent[rng.integers(0, 5, n)] + 0.1 * rng.standard_normal((n, d))).astype(np.float32)
    ix = sivf.Index(d, 5, cent, slab_capacity=8, num_slabs=n, id_capacity=n, max_batch=n, max_queries=64, max_k=8, max_nprobe=5)
    ref = oracle.OracleIndex(d, 5, cent, 0, 8, n, n)
    ix.add(x, np.arange(n))
    assert ix.sync() == 0 and ref.add(x, np.arange(n)) == 0
    np.testing.assert_array_equal(ix.get_rows(np.arange(n)).cpu().numpy(), x)
    gd, gl = ix.search(x[-64:], 8, 5)
    assert ix.sync() == 0
    st, rd, rl = ref.search(x[-64:], 8, 5)
    assert st == 0 and compare_results(gd.cpu().numpy(), gl.cpu().numpy(), rd, rl) == 0
