// Search over the slab-resident lists (the paper's Sec. 3.3 / Alg. 3,
// re-designed for wave64 and query batches).
//
// The paper gives one warp to one query and walks each probed chain per
// query.  Here the (query, probed list) pairs of a whole batch are inverted
// to list-major work items: an item is one list and a tile of up to T queries
// that probe it.  One wave scans the list's slabs once per item (lane <->
// slot, 64 slots per step, coalesced 1 KiB loads), computing the canonical
// FP32 distance of every slot to all T queries of the tile, which sit in LDS.
// Each query keeps its best kcap (distance, id) keys sorted across the lanes
// of the wave; candidates below the current k-th key are inserted with
// ballots and lane shifts.  A final kernel merges the per-list partial
// results of each query.
//
//   k_inv_count   rank of each (query, probe) pair within its list (or
//                 k_inv_count_lds: block histograms, fewer global atomics)
//   k_inv_plan    per-list pair offsets, chunks, item offsets
//   k_inv_fill    work items (list, tile, chunk); pair ids grouped by list
//   (k_inv_small  the three in one launch, for small batches)
//   k_scan        one wave per item: distances + per-query top-kcap
//   k_merge       one wave per query: kcap-way merge of its probe partials
#include "scan_dev.h"

namespace sivf {


// Whether query qi belongs to the pass of class c.
__device__ __forceinline__ bool in_class(const KClass &c, int qi) {
    if (c.lo < 0 && c.hi == 0x7FFFFFFF) return true;
    int kq = c.kpq ? c.kpq[qi] : c.k;
    kq = kq < 0 ? 0 : (kq > c.k ? c.k : kq);
    return kq > c.lo && kq <= c.hi;
}

// List of pair p, or -1 when it probes nothing or its query is outside the pass.
__device__ __forceinline__ int pair_list(const int32_t *probes, int p, const KClass &c) {
    const int l = probes[p], qi = p / c.np_stride, j = p - qi * c.np_stride;
    return (l >= 0 && j >= c.plo && j < c.phi && in_class(c, qi)) ? l : -1;
}

__global__ __launch_bounds__(256) void k_inv_count(Dev S, int npairs, const int32_t *__restrict__ probes,
                                                   int32_t *__restrict__ pair_rank, KClass cls, int nq,
                                                   uint32_t *__restrict__ gthr) {
    const int p = blockIdx.x * 256 + threadIdx.x;
    if (p < nq) gthr[p] = 0xFFFFFFFFu;   // no key published yet
    const bool active = p < npairs;
    const int l = active ? pair_list(probes, p, cls) : -1;
    const bool act = l >= 0;
    const int r = act ? atomicAdd(&S.l_qc[l], 1) : 0;   // a wave's 64 pairs hit ~64 distinct lists
    if (active) pair_rank[p] = act ? r : -1;
}

// The same ranks with one device-scope atomic per (block, list) instead of
// one per pair: a block of 1024 threads takes INV_PB pairs, ranks them
// within the block by LDS atomics on a per-list histogram (nlist ints of
// dynamic LDS), reserves each list's block total with one atomic on l_qc,
// and adds that base.  Used when the histogram fits in 64 KiB.
constexpr int INV_PB = 8192;
__global__ __launch_bounds__(1024) void k_inv_count_lds(Dev S, int npairs, const int32_t *__restrict__ probes,
                                                        int32_t *__restrict__ pair_rank, KClass cls, int nq,
                                                        uint32_t *__restrict__ gthr) {
    extern __shared__ int32_t hist[];
    const int tid = threadIdx.x;
    for (int i = blockIdx.x * 1024 + tid; i < nq; i += gridDim.x * 1024) gthr[i] = 0xFFFFFFFFu;   // none published yet
    const int64_t p0 = (int64_t)blockIdx.x * INV_PB;
    const int n = (int)min((int64_t)INV_PB, (int64_t)npairs - p0);
    for (int i = tid; i < S.nlist; i += 1024) hist[i] = 0;
    __syncthreads();
    for (int i = tid; i < n; i += 1024) {
        const int l = pair_list(probes, (int)(p0 + i), cls);
        pair_rank[p0 + i] = l >= 0 ? atomicAdd(&hist[l], 1) : -1;
    }
    __syncthreads();
    for (int i = tid; i < S.nlist; i += 1024) {
        const int c = hist[i];
        if (c > 0) hist[i] = atomicAdd(&S.l_qc[i], c);
    }
    __syncthreads();
    for (int i = tid; i < n; i += 1024) {
        const int r = pair_rank[p0 + i];
        if (r >= 0) pair_rank[p0 + i] = r + hist[probes[p0 + i]];
    }
}

// Block sums of two int64 values (every thread gets both totals).
__device__ __forceinline__ void block_sum2(long long &a, long long &b, long long *sred) {
    for (int o = 32; o > 0; o >>= 1) {
        a += __shfl_xor(a, o);
        b += __shfl_xor(b, o);
    }
    const int w = threadIdx.x >> 6, nw = blockDim.x >> 6;
    __syncthreads();
    if (lane_id() == 0) {
        sred[w] = a;
        sred[16 + w] = b;
    }
    __syncthreads();
    a = 0;
    b = 0;
    for (int i = 0; i < nw; i++) {
        a += sred[i];
        b += sred[16 + i];
    }
}


// Chunk of a search whose scan costs `cost` (list positions x query tiles of T):
// log2 of the positions per work item, at most sh0.  FILL_ITEMS work items
// fill the chip once (12 waves on each of 256 CUs); a batch with fewer than that at
// sh0 gets shorter chunks.  VALU scans (T < 16) have no start-up worth keeping
// long chunks for: at least FILL_ITEMS items, down to 2 steps of 64 positions
// (1 query, 32 lists of about 2,500: 333 us in 32 items, 16 in 640).  The
// matrix-core scans pay for every work item's cold start (no threshold yet: a
// bisection, and the exact distances of the first candidates) about what eight
// steps cost: at most half of FILL_ITEMS items, of four steps or more
// (3,277 queries x 6 lists of 1,000 x 32 values: 260 us unsplit, 322 us in chunks
// of 256).  A larger batch on them gets chunks of 2^13, while those are at most
// 8 FILL_ITEMS: a very long list otherwise ends long after the others (3,854
// queries with k up to 100 on lists of 400 to 300,000: 5.4 ms at 2^14, 4.5 ms at
// 2^13).
__device__ __forceinline__ int plan_shift(long long cost, int sh0, int T) {
    auto flog2 = [](long long v) { return v <= 1 ? 0 : 63 - __clzll(v); };
    const int fill = flog2(cost / FILL_ITEMS);
    const int s = T < 16 ? max(fill, 7) : max(min(max(fill + 2, 8), 13), flog2(cost / (8 * FILL_ITEMS)) + 1);
    return min(s, sh0);
}

// One block of 1,024 threads plans the whole search:
//  1. snapshot every list's length (the scan reads only these entries; a
//     second pass of the same search keeps the first pass's snapshot) and
//     lay out the (query, probe) pairs list by list;
//  2. split lists into chunks of 2^sh positions (plan_shift), with the smallest
//     sh from there up whose partial results (one per pair and chunk) and work
//     items (one per tile of T pairs and chunk) fit their buffers;
//  3. per-list offsets of partial slots and items; reset the work counters;
//  4. cut the items into 8 ranges, one per XCD, of equal scan cost (list
//     positions x query tiles) -- equal item counts leave XCDs idle while
//     others finish long lists -- each at most xcd_cap items (the blocks an
//     XCD receives in the dispatch schedule).
// Wave w holds lists 64 E w + 64 e + lane, e < E, in registers, so every array is
// read once, coalesced, and the four prefix sums take one DPP scan per 64 lists
// and one exchange between the waves.  What bounds it is latency on one CU: at
// 16,384 lists a loop of block-wide scans over 1,024 lists at a time took 101 us.
struct PlanShared {
    int wt[4][16];
    long long red[32];
    int xb[9];
};

// Totals of four values over the block's waves, and each wave's exclusive sums.
__device__ __forceinline__ void wave_offsets4(int (&v)[4], int (&before)[4], int (&total)[4], PlanShared &sm) {
    const int w = threadIdx.x >> 6;
#pragma unroll
    for (int i = 0; i < 4; i++) {
        int x = v[i];
        for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o);
        if (lane_id() == 0) sm.wt[i][w] = x;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 4; i++) {
        before[i] = total[i] = 0;
        for (int j = 0; j < 16; j++) {
            const int x = sm.wt[i][j];
            before[i] += j < w ? x : 0;
            total[i] += x;
        }
    }
}

// qc, len: pairs and snapshot length of this thread's lists.  qoff_l, ioff_l (or
// NULL): copies of the pair and item offsets in LDS.  Returns the item count.
template <int E>
__device__ __forceinline__ int plan_core(const Dev &S, int T, int sh0, int64_t slot_cap, int64_t item_cap,
                                         int xcd_cap, const int (&qc)[E], const int (&len)[E], int *qoff_l,
                                         int *ioff_l, PlanShared &sm) {
    const int lane = lane_id(), l0 = (threadIdx.x >> 6) * 64 * E + lane;
    long long cost = 0, none = 0;
#pragma unroll
    for (int e = 0; e < E; e++) cost += qc[e] > 0 ? (long long)cdiv_s(qc[e], T) * len[e] : 0;
    block_sum2(cost, none, sm.red);
    int sh = plan_shift(cost, sh0, T);
    for (;;) {
        long long slots = 0, items = 0;
#pragma unroll
        for (int e = 0; e < E; e++) {
            const int nc = qc[e] > 0 ? list_chunks(len[e], sh) : 0;
            slots += (long long)qc[e] * nc;
            items += (long long)cdiv_s(qc[e], T) * nc;
        }
        block_sum2(slots, items, sm.red);
        if ((slots <= slot_cap && items <= item_cap) || sh >= 31) break;   // sh = 31: one chunk per list
        sh++;
    }
    // costs in units that keep their sum below 2^30 (the cuts need no more)
    const int cb = max(0, 34 - (int)__clzll(cost));
    auto values = [&](int e, int (&v)[4]) {
        const int nc = qc[e] > 0 ? list_chunks(len[e], sh) : 0, nt = cdiv_s(qc[e], T);
        v[0] = qc[e];
        v[1] = qc[e] * nc;
        v[2] = nt * nc;
        v[3] = nc > 0 ? (int)(((long long)nt * len[e]) >> cb) : 0;
    };
    int sum[4] = {0, 0, 0, 0}, carry[4], total[4];
#pragma unroll
    for (int e = 0; e < E; e++) {
        int v[4];
        values(e, v);
#pragma unroll
        for (int i = 0; i < 4; i++) sum[i] += v[i];
    }
    if (threadIdx.x < 9) sm.xb[threadIdx.x] = -1;
    wave_offsets4(sum, carry, total, sm);
#pragma unroll
    for (int e = 0; e < E; e++) {
        const int l = l0 + 64 * e;
        int v[4], ex[4];
        values(e, v);
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const int incl = wave_incl_scan_dpp(v[i]);
            ex[i] = carry[i] + incl - v[i];
            carry[i] += readlane_i(incl, 63);
        }
        if (l < S.nlist) {
            S.l_qoff[l] = ex[0];
            S.l_pbase[l] = ex[1];
            S.l_ioff[l] = ex[2];
            S.l_qcs[l] = qc[e];
            if (qoff_l) {
                qoff_l[l] = ex[0];
                ioff_l[l] = ex[2];
            }
            // XCD boundary x (1..7) at cost x * W / 8 falls in this list's [ex, ex + v)
            for (int x = 1; x < 8 && v[3] > 0; x++) {
                const int target = (int)((long long)total[3] * x / 8);
                if (target >= ex[3] && target < ex[3] + v[3])
                    sm.xb[x] = ex[2] + (int)((double)(target - ex[3]) / (double)v[3] * v[2]);
            }
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        const int n = total[2];
        // boundaries not hit (zero-cost tail) follow the previous one; then cap every range
        int b = 0;
        S.ctl[CTL_XB] = 0;
        for (int x = 1; x < 8; x++) {
            int t = sm.xb[x] < 0 ? b : sm.xb[x];
            t = t < b ? b : t;
            t = t > b + xcd_cap ? b + xcd_cap : t;               // this range fits its XCD's blocks
            const int rest = n - (8 - x) * xcd_cap;               // the later ranges must fit too
            t = t < rest ? rest : t;
            t = t > n ? n : t;
            S.ctl[CTL_XB + x] = t;
            b = t;
        }
        S.ctl[CTL_XB + 8] = n;
        S.ctl[CTL_NITEMS] = n;
        S.ctl[CTL_CHUNK] = sh;
    }
    if (threadIdx.x < 8) S.ctl[CTL_WORK0 + CTL_WORK_STRIDE * threadIdx.x] = 0;
    return total[2];
}

// Length of list l as this pass scans it, and the probe count per list (host
// tier: the coldest lists are offloaded first), saturating.
__device__ __forceinline__ int plan_len(const Dev &S, int l, int qc, int snap, int32_t *heat) {
    int len;
    if (snap) {
        len = S.len[l];
        S.l_snap[l] = len;
    } else {
        len = S.l_snap[l];
    }
    if (heat && qc > 0) heat[l] = (int32_t)min((int64_t)heat[l] + qc, (int64_t)0x7FFFFFFF);
    return len;
}

template <int E>
__global__ __launch_bounds__(1024) void k_inv_plan(Dev S, int T, int sh0, int64_t slot_cap, int64_t item_cap,
                                                   int xcd_cap, int snap, int32_t *__restrict__ heat) {
    __shared__ PlanShared sm;
    const int l0 = (threadIdx.x >> 6) * 64 * E + lane_id();
    int qc[E], len[E];
#pragma unroll
    for (int e = 0; e < E; e++) {
        const int l = l0 + 64 * e;
        qc[e] = l < S.nlist ? S.l_qc[l] : 0;
        len[e] = l < S.nlist ? plan_len(S, l, qc[e], snap, heat) : 0;
        if (l < S.nlist) S.l_qc[l] = 0;
    }
    plan_core<E>(S, T, sh0, slot_cap, item_cap, xcd_cap, qc, len, nullptr, nullptr, sm);
}

// The rest of the plan, on as many blocks as it takes: the first item_blocks
// blocks list each list's work items, chunk-major (consecutive items read the
// same slabs for different query tiles), one wave per list; the others group the
// pairs by list.
__global__ __launch_bounds__(256) void k_inv_fill(Dev S, int T, int item_blocks, int npairs,
                                                  const int32_t *__restrict__ probes,
                                                  const int32_t *__restrict__ pair_rank,
                                                  int32_t *__restrict__ list_pairs, int32_t *__restrict__ item_list,
                                                  int32_t *__restrict__ item_tile, int32_t *__restrict__ item_chunk) {
    if ((int)blockIdx.x >= item_blocks) {
        const int p = ((int)blockIdx.x - item_blocks) * 256 + threadIdx.x;
        const int r = p < npairs ? pair_rank[p] : -1;
        if (r >= 0) list_pairs[S.l_qoff[probes[p]] + r] = p;
        return;
    }
    const int l = blockIdx.x * 4 + (threadIdx.x >> 6), lane = lane_id();
    if (l >= S.nlist) return;
    const int qc = S.l_qcs[l];
    if (qc == 0) return;
    const int nc = list_chunks(S.l_snap[l], S.ctl[CTL_CHUNK]);
    const int nt = cdiv_s(qc, T);
    const int base = S.l_ioff[l];
    for (int i = lane; i < nt * nc; i += 64) {
        item_list[base + i] = l;
        item_chunk[base + i] = i / nt;
        item_tile[base + i] = i % nt;
    }
}

// The whole plan in one launch, for at most SP_PAIRS pairs on at most SP_LISTS
// lists: ranks from an LDS histogram, then plan_core, then pairs and items from
// the offsets in LDS (an item finds its list by bisection).  A launch that finds
// the previous one's results costs about 4.5 us here, more than the work of any of
// the five kernels it replaces (count, plan, items, pairs, threshold fill).
constexpr int SP_PAIRS = 8192, SP_LISTS = 4096, SP_E = SP_LISTS / 1024;
__global__ __launch_bounds__(1024) void k_inv_small(Dev S, int T, int sh0, int64_t slot_cap, int64_t item_cap,
                                                    int xcd_cap, int snap, int32_t *__restrict__ heat, int nq,
                                                    int npairs, const int32_t *__restrict__ probes,
                                                    int32_t *__restrict__ pair_rank, int32_t *__restrict__ list_pairs,
                                                    int32_t *__restrict__ item_list, int32_t *__restrict__ item_tile,
                                                    int32_t *__restrict__ item_chunk, KClass cls,
                                                    uint32_t *__restrict__ gthr) {
    extern __shared__ int32_t lds[];   // pairs per list, then pair offsets, then item offsets (nlist each)
    __shared__ PlanShared sm;
    int32_t *hist = lds, *qoff = lds + S.nlist, *ioff = lds + 2 * S.nlist;
    const int tid = threadIdx.x;
    for (int i = tid; i < nq; i += 1024) gthr[i] = 0xFFFFFFFFu;   // no key published yet
    for (int i = tid; i < S.nlist; i += 1024) hist[i] = 0;
    int pl[SP_PAIRS / 1024], pr[SP_PAIRS / 1024];
#pragma unroll
    for (int i = 0; i < SP_PAIRS / 1024; i++) {
        const int p = tid + 1024 * i;
        pl[i] = p < npairs ? pair_list(probes, p, cls) : -1;
    }
    const int l0 = (tid >> 6) * 64 * SP_E + lane_id();
    int qc[SP_E], len[SP_E];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < SP_PAIRS / 1024; i++) pr[i] = pl[i] >= 0 ? atomicAdd(&hist[pl[i]], 1) : -1;
    __syncthreads();
#pragma unroll
    for (int e = 0; e < SP_E; e++) {
        const int l = l0 + 64 * e;
        qc[e] = l < S.nlist ? hist[l] : 0;
        len[e] = l < S.nlist ? plan_len(S, l, qc[e], snap, heat) : 0;
    }
    const int n = plan_core<SP_E>(S, T, sh0, slot_cap, item_cap, xcd_cap, qc, len, qoff, ioff, sm);
    // plan_core's last barrier is behind its LDS writes
#pragma unroll
    for (int i = 0; i < SP_PAIRS / 1024; i++) {
        const int p = tid + 1024 * i;
        if (p < npairs) pair_rank[p] = pr[i];
        if (pr[i] >= 0) list_pairs[qoff[pl[i]] + pr[i]] = p;
    }
    for (int i = tid; i < n; i += 1024) {
        int lo = 0, hi = S.nlist - 1;   // the last list whose first item is at most i holds it
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (ioff[mid] <= i) lo = mid;
            else hi = mid - 1;
        }
        const int nt = cdiv_s(hist[lo], T), j = i - ioff[lo];
        item_list[i] = lo;
        item_chunk[i] = j / nt;
        item_tile[i] = j % nt;
    }
}

// Distances of 64 consecutive list positions (lane <-> slot) to the T queries
// of a tile, in the canonical order (dimensions ascending, one fma each), then
// offered to each query's top-k.  QV(t, c) gives query t's dimension chunk c.
// Where there are more items than the chip runs at once, lane t (t < nt, query qg)
// reads the best k-th key that finished items have published for its query, and
// publishes this item's at its end: a candidate behind it cannot be a result, so an
// item scanned late sorts few keys of its own and the merge reads fewer (1,000 queries
// x 16 of 1,024 lists, 500k x 128: the step 544 -> 527 us).  Read at every 64 rows it
// costs more than it saves (200 us instead of 60 for 100 queries x 16), and so it does
// where all items run at once (37 queries x 16: 60 -> 63 us).
#define SIVF_SCAN_RANGE(QV)                                                                      \
    const int cs_ = __builtin_ctz(C), cm_ = C - 1; /* slab capacities are powers of two */       \
    const int nslab = (len + cm_) >> cs_;                                                        \
    int wbase = -(1 << 30), wslab = 0; /* lane j holds the slab of ordinal wbase + j */          \
    const bool share_ = S.ctl[CTL_XB + 8] > 2 * FILL_ITEMS;                                      \
    const uint32_t pub = share_ && lane < nt ? __hip_atomic_load(gthr + qg, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : ~0u; \
    for (int base = p0; base < p1; base += 64) {                                                 \
        const int p = base + lane;                                                               \
        const bool valid = p < p1;                                                               \
        const int pc = valid ? p : p1 - 1;                                                       \
        const int last_ord = min(base + 63, p1 - 1) >> cs_;                                      \
        if (last_ord >= wbase + 64) {                                                            \
            wbase = base >> cs_;                                                                 \
            wslab = (wbase + lane < nslab) ? slab_of(S, l, wbase + lane) : 0;                    \
        }                                                                                        \
        const int slab = __shfl(wslab, (pc >> cs_) - wbase);                                     \
        const int slot = pc & cm_;                                                               \
        /* lazy deletes: a slot whose validity bit is clear holds no entry */                    \
        const bool live_ = valid && (!S.bits || ((valid_word(S, slab, slot) >> (slot & 63)) & 1ull)); \
        const float4 *xp = S.data + (int64_t)slab * dp4 * C + slot;                              \
        float acc[T];                                                                            \
        _Pragma("unroll") for (int t = 0; t < T; t++) acc[t] = 0.f;                              \
        _Pragma("unroll UNR") for (int c = 0; c < dp4; c++) {                                    \
            const float4 xv = xp[(int64_t)c * C];                                                \
            _Pragma("unroll") for (int t = 0; t < T; t++) {                                      \
                const float4 qv = QV(t, c);                                                      \
                if (METRIC == 0) {                                                               \
                    float e;                                                                     \
                    e = qv.x - xv.x;                                                             \
                    acc[t] = __builtin_fmaf(e, e, acc[t]);                                       \
                    e = qv.y - xv.y;                                                             \
                    acc[t] = __builtin_fmaf(e, e, acc[t]);                                       \
                    e = qv.z - xv.z;                                                             \
                    acc[t] = __builtin_fmaf(e, e, acc[t]);                                       \
                    e = qv.w - xv.w;                                                             \
                    acc[t] = __builtin_fmaf(e, e, acc[t]);                                       \
                } else {                                                                         \
                    acc[t] = __builtin_fmaf(qv.x, xv.x, acc[t]);                                 \
                    acc[t] = __builtin_fmaf(qv.y, xv.y, acc[t]);                                 \
                    acc[t] = __builtin_fmaf(qv.z, xv.z, acc[t]);                                 \
                    acc[t] = __builtin_fmaf(qv.w, xv.w, acc[t]);                                 \
                }                                                                                \
            }                                                                                    \
        }                                                                                        \
        const uint32_t id = S.sids[(int64_t)slab * C + slot];                                    \
        _Pragma("unroll") for (int t = 0; t < T; t++) {                                          \
            K.thr[t] = min(K.thr[t], (uint32_t)__builtin_amdgcn_readlane(pub, t));               \
            if (t < nt) topk_offer(K, t, live_, key_hi<METRIC>(acc[t]), id, buf, skq, kcap);     \
        }                                                                                        \
    }                                                                                            \
    SIVF_ITEM_SLOT(T)                                                                            \
    _Pragma("unroll") for (int t = 0; t < T; t++) {                                              \
        if (t < nt) {                                                                            \
            if (K.cnt[t] > 0) topk_flush(K, t, buf, skq, kcap);                                  \
            uint64_t *dst = partials + (slot0 + (int64_t)t * nc) * kcap;                         \
            if (lane < kcap) dst[lane] = K.top[t];                                               \
            if (WIDE && lane + 64 < kcap) dst[64 + lane] = K.top2[WIDE ? t : 0];                 \
        }                                                                                        \
    }                                                                                            \
    uint32_t mine = ~0u;                                                                         \
    _Pragma("unroll") for (int t = 0; t < T; t++) mine = lane == t ? K.thr[t] : mine;            \
    if (share_ && lane < nt && mine < pub && skq[lane & (T - 1)] > 0)                                                   \
        __hip_atomic_fetch_min(gthr + qg, mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);


// Dimension chunks in flight per lane.  The fewer queries share a chunk, the
// less VALU work covers its load, and the more registers are free for loads: T x
// unroll = 16.  1,000 queries on 96-entry tiles of 960-value rows, T = 4: 335 us
// with two chunks in flight, 267 with four.
constexpr int scan_unroll(int T) { return 16 / T; }

// Queries come straight from the caller's rows with wave-uniform addresses,
// so the compiler reads them through the scalar cache into SGPRs and every
// VALU op takes its query operand from an SGPR (no LDS traffic).  Needs
// d % 4 == 0 and 16-byte aligned rows.
template <int T, int METRIC, bool WIDE, bool PERS>
__global__ __launch_bounds__(64) void k_scan_sq(Dev S, const int32_t *__restrict__ item_list,
                                                const int32_t *__restrict__ item_tile,
                                                const int32_t *__restrict__ item_chunk,
                                                const int32_t *__restrict__ list_pairs,
                                                const float *__restrict__ q, int np_stride, int kcap, int k,
                                                const int32_t *__restrict__ kpq, uint64_t *__restrict__ partials,
                                                uint32_t *__restrict__ gthr) {
    __shared__ uint64_t buf[T * 64];
    __shared__ int skq[T];
    const int lane = threadIdx.x;
    const int dp4 = S.dp4, C = S.C, sh = S.ctl[CTL_CHUNK];
    SIVF_ITEM_LOOP_BEGIN
    SIVF_ITEM_DECODE(T)
    constexpr int UNR = scan_unroll(T);
    const float4 *qrow[T];
    TopK<T, WIDE> K;
#pragma unroll
    for (int t = 0; t < T; t++) {
        const int pr = pairs[t < nt ? t : 0];
        qrow[t] = reinterpret_cast<const float4 *>(q + (int64_t)(pr / np_stride) * S.d);
    }
    __syncthreads();
    const int qg = pairs[lane < nt ? lane : 0] / np_stride;
    if (lane < T) skq[lane] = lane < nt ? query_k(kpq, k, qg) : 0;
    __syncthreads();
    topk_init(K, skq);
#define SIVF_QV_SQ(t, c) qrow[t][c]
    SIVF_SCAN_RANGE(SIVF_QV_SQ)
#undef SIVF_QV_SQ
    SIVF_ITEM_LOOP_END
}

// General path: query rows of any alignment or dimension, staged in LDS.
template <int T, int METRIC, bool WIDE, bool PERS>
__global__ __launch_bounds__(64) void k_scan(Dev S, const int32_t *__restrict__ item_list,
                                             const int32_t *__restrict__ item_tile,
                                             const int32_t *__restrict__ item_chunk,
                                             const int32_t *__restrict__ list_pairs, const float *__restrict__ q,
                                             int np_stride, int kcap, int k, const int32_t *__restrict__ kpq,
                                             uint64_t *__restrict__ partials, uint32_t *__restrict__ gthr) {
    extern __shared__ float4 sq[];   // [T][dp4]
    __shared__ uint64_t buf[T * 64];
    __shared__ int skq[T];
    const int lane = threadIdx.x;
    const int dp4 = S.dp4, C = S.C, d = S.d, sh = S.ctl[CTL_CHUNK];
    SIVF_ITEM_LOOP_BEGIN
    SIVF_ITEM_DECODE(T)
    constexpr int UNR = scan_unroll(T);
    TopK<T, WIDE> K;
    __syncthreads();
    for (int t = 0; t < T; t++) {
        const int pr = t < nt ? pairs[t] : -1;
        const float *qr = q + (int64_t)(pr < 0 ? 0 : pr / np_stride) * d;
        for (int c = lane; c < dp4; c += 64) {
            float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
            if (pr >= 0) {
                const int j = 4 * c;
                v.x = j < d ? qr[j] : 0.f;
                v.y = j + 1 < d ? qr[j + 1] : 0.f;
                v.z = j + 2 < d ? qr[j + 2] : 0.f;
                v.w = j + 3 < d ? qr[j + 3] : 0.f;
            }
            sq[t * dp4 + c] = v;
        }
    }
    const int qg = pairs[lane < nt ? lane : 0] / np_stride;
    if (lane < T) skq[lane] = lane < nt ? query_k(kpq, k, qg) : 0;
    __syncthreads();
    topk_init(K, skq);
#define SIVF_QV_LDS(t, c) sq[(t) * dp4 + (c)]
    SIVF_SCAN_RANGE(SIVF_QV_LDS)
#undef SIVF_QV_LDS
    SIVF_ITEM_LOOP_END
}

#undef SIVF_SCAN_RANGE

// The best keys of each query's partial lists (one per probe and chunk,
// sorted, kcap long), by WPQ waves per query.  The lists are numbered probe after
// probe, 64 probes at a time; each lane takes one list of a round of 64, reads it
// four keys at a time and leaves it at the first key above the bound; keys up to
// the bound are queued in LDS and merged 64 at a time into the sorted result
// (bitonic network), whose kq-th key is the new bound.  The bound starts at the
// value the scan's work items published for the query (gthr; the kq best keys are
// at or below it), so few keys of most lists are read at all.  What bounds it is the
// chain of dependent reads, one or two per round of lists, not kq rounds of a
// k-way merge: 40 keys of 40 lists per query (477 queries) took 38 us with one
// key per round and takes 14.  The waves of a query take its rounds in turn
// and the first merges their results: WPQ = 4 where the queries alone leave
// the chip idle (few queries, their lists split into many chunks).
// k: the call's k; each query keeps kmul * (its k) results, at most out_stride
// (the row stride of dist / labels, <= 128).  prior (or NULL): one more sorted
// source per query, prior_stride keys (~0 padded) -- the host tier's results;
// keys_out (or NULL): write the sorted keys there (stride out_stride, ~0
// padded) instead of dist / labels.
constexpr int MG_BUF = 64 + 4 * 64;   // a round adds at most 4 keys per lane to fewer than 64 waiting ones
template <bool WIDE, int WPQ>
__global__ __launch_bounds__(256) void k_merge(Dev S, int nq, int np_stride, const int32_t *__restrict__ probes,
                                               const int32_t *__restrict__ pair_rank,
                                               const uint64_t *__restrict__ partials, int kcap, int out_stride,
                                               int k, int kmul, const int32_t *__restrict__ kpq,
                                               float *__restrict__ dist, int64_t *__restrict__ labels, KClass cls,
                                               uint32_t *__restrict__ gthr,
                                               const uint64_t *__restrict__ prior, int prior_stride,
                                               uint64_t *__restrict__ keys_out) {
    __shared__ uint64_t sbuf[4][MG_BUF];
    const int w = threadIdx.x >> 6, lane = lane_id();
    const int sub = w % WPQ;   // this wave's turn among the query's waves
    const int qi = blockIdx.x * (4 / WPQ) + w / WPQ;
    // a query of another pass: its results come from that one (a query's waves leave together, and with
    // WPQ > 1 they are the whole block)
    if (qi >= nq || !in_class(cls, qi)) return;
    const int sh = S.ctl[CTL_CHUNK];
    int kq = kpq ? kpq[qi] : k;
    kq = kq < 0 ? 0 : (kq > k ? k : kq);
    kq = min(kq * kmul, out_stride);
    uint64_t *buf = sbuf[w];
    uint64_t res = ~0ull, res2 = ~0ull;   // result r sits in lane r (r < 64) or lane r - 64 of res2
    // keys above the bound are not among the kq best
    uint64_t bound = gthr ? ((uint64_t)gthr[qi] << 32) | 0xFFFFFFFFull : ~0ull;
    auto take = [&](uint64_t b) {   // 64 more keys (~0: none)
        if (WIDE) merge128_with(res, res2, b);
        else res = merge_sorted_with(res, b);
        const uint64_t kth = (WIDE && kq > 64) ? readlane_u64(res2, kq - 65) : readlane_u64(res, kq - 1);
        bound = kth < bound ? kth : bound;
    };
    if (kq > 0) {
        if (prior && sub == 0) {
            const uint64_t *pr = prior + (int64_t)qi * prior_stride;
            for (int i = 0; i < prior_stride; i += 64) take(i + lane < prior_stride ? pr[i + lane] : ~0ull);
        }
        const int32_t *prow = probes + (int64_t)qi * np_stride;
        const int32_t *rrow = pair_rank + (int64_t)qi * np_stride;
        int nb = 0;      // keys waiting in buf (wave-uniform)
        int round = 0;
        for (int p0 = 0; p0 < np_stride; p0 += 64) {
            const int p = p0 + lane;
            const int l = p < np_stride ? prow[p] : -1;
            const int rank = l >= 0 ? rrow[p] : -1;   // -1: a pair of another phase
            const int nc = rank >= 0 ? list_chunks(S.l_snap[l], sh) : 0;
            const int64_t slot = nc > 0 ? (int64_t)S.l_pbase[l] + (int64_t)rank * nc : 0;
            const int incl = wave_incl_scan_dpp(nc);
            const int total = readlane_i(incl, 63), excl = incl - nc;
            for (int s0 = 0; s0 < total; s0 += 64) {
                if (WPQ > 1 && (round++ % WPQ) != sub) continue;
                // list s0 + lane: its probe is the last lane whose exclusive sum is at most it (empty
                // probes share their sum with the next one)
                const int s = s0 + lane;
                int at = 0;
#pragma unroll
                for (int step = 32; step > 0; step >>= 1) {
                    const int e = __shfl(excl, at + step);
                    if (e <= s) at += step;
                }
                const int64_t base = ((int64_t)__shfl((int)(slot >> 32), at) << 32) | (uint32_t)__shfl((int)slot, at);
                const uint64_t *src = partials + (base + (s - __shfl(excl, at))) * kcap;
                bool open = s < total;
                int j = 0;   // next key
                while (ballot(open)) {
                    uint64_t v[4] = {~0ull, ~0ull, ~0ull, ~0ull};
                    if (open) {   // kcap is a multiple of 16: four keys, 32-byte aligned
                        const ulonglong2 a = *reinterpret_cast<const ulonglong2 *>(src + j);
                        const ulonglong2 b = *reinterpret_cast<const ulonglong2 *>(src + j + 2);
                        v[0] = a.x;
                        v[1] = a.y;
                        v[2] = b.x;
                        v[3] = b.y;
                    }
#pragma unroll
                    for (int i = 0; i < 4; i++) {
                        const bool pass = v[i] <= bound && v[i] != ~0ull;
                        const uint64_t m = ballot(pass);
                        if (pass) buf[nb + (int)__builtin_popcountll(m & lanemask_lt())] = v[i];
                        nb += (int)__builtin_popcountll(m);
                    }
                    j += 4;
                    if (v[3] > bound || v[3] == ~0ull || j >= kcap) open = false;
                    __builtin_amdgcn_wave_barrier();
                    while (nb >= 64) {
                        nb -= 64;
                        take(buf[nb + lane]);
                        __builtin_amdgcn_wave_barrier();
                    }
                }
            }
        }
        if (nb > 0) take(lane < nb ? buf[lane] : ~0ull);
    }
    if (WPQ > 1) {   // the other waves' results join the first's
        __builtin_amdgcn_wave_barrier();
        buf[lane] = res;
        if (WIDE) buf[64 + lane] = res2;
        __syncthreads();
        if (sub != 0) return;
        if (kq > 0) {
            for (int o = 1; o < WPQ; o++) {
                take(sbuf[w + o][lane]);
                if (WIDE) take(sbuf[w + o][64 + lane]);
            }
        }
    }
    if (keys_out && gthr && kq > 0) {   // the merged k-th key bounds what the next phase can add
        const uint64_t kth = (WIDE && kq > 64) ? readlane_u64(res2, kq - 65) : readlane_u64(res, kq - 1);
        if (lane == 0 && kth != ~0ull) gthr[qi] = (uint32_t)(kth >> 32);
    }
    for (int h = 0; h < 2; h++) {
        const int r = lane + 64 * h;
        if (r < out_stride) {
            const uint64_t key = h ? res2 : res;
            const int64_t o = (int64_t)qi * out_stride + r;
            if (keys_out) {
                keys_out[o] = r < kq ? key : ~0ull;
            } else if (r < kq && key != ~0ull) {
                dist[o] = key_value(key, S.metric);
                labels[o] = (int64_t)(uint32_t)key;
            } else {
                dist[o] = S.metric == 0 ? __int_as_float(0x7F800000) : __int_as_float((int)0xFF800000);
                labels[o] = -1;
            }
        }
    }
}

// Default queries per tile (the LDS path holds T * ceil(d/4) * 16 bytes,
// within 32 KiB).  Measured on the window workload: T=8 with two dimension
// chunks in flight beats T=16, whose query operands no longer fit the SGPR
// file.  The MFMA scan's tile is one 16-column operand.
int default_tile(int storage, int d, int C, int kcap) {
    if (storage != 0 || cert_ok(storage, d, C, kcap)) return 16;
    return d <= 1024 ? 8 : 4;
}

// Queries per work item of a search without a schedule of the caller's own, by
// the pairs per list (each list is probed by about that many of the batch's
// queries).  A tile of 16 on the matrix cores costs the same for one query as for
// 16, and its threshold and exact recomputation start cold in every work item;
// the VALU scan reads a list once per 2 or 4 queries.  Scan times in us at
// 2, 4 and 16 queries per tile (1M x 128, 1,024 lists, 32 probes): 1 query
// 16, 20, 40; 64 queries (2 pairs per list) 85, 90, 422; 200 (6 per list) -, 188,
// 388; 500 (16 per list) -, 435, 413; 1,000 (31 per list) -, 699, 520.  On
// 200k x 128 with 6 pairs per list 57, 62, 141.  For the pass of queries with k > 64
// the matrix-core scan has to insert up to 128 keys per query and work item
// one at a time, and pays off later (1M x 128 at k = 100, 1,024 lists, 4 and 16 per
// tile: 98 pairs per list 0.58 to 1.17 times as fast by data, 195 and up 1.1 to 2.4
// times for 8 of 9, 0.92 for one; mixed batches, where a third has k = 100 and all
// are counted, by half their pairs: 187 per list 3.4 against 6.2 ms, 2,000 28 against
// 20 ms).  Wide rows (no matrix-core scan) take 4 rather than 8: 267 against
// 374 us at 31 pairs per list of 960 values, 776 against 970 at 125.
int auto_tile(const Dev &S, int64_t npairs, bool deep) {
    if (S.storage != 0) return 16;
    if (npairs <= 6ll * S.nlist) return 2;
    if (S.tile != 16 || npairs <= (deep ? 200ll : 16ll) * S.nlist) return 4;
    return 16;
}

int search_tile(const Dev &S) { return S.tile; }

// Exact FP32 re-rank: one wave per query; lane i recomputes the canonical
// FP32 distance of candidate i from the fp32 shadow row, then the wave sorts
// the keys and keeps the query's k best.  A row's 16-byte chunks lie C slots
// apart, so a large batch is bound by the lines its gathers touch (16,000 queries x
// 40 rows of 96 values: 0.3 ms), a small one by the latency of a lane's loads:
// eight are in flight at once and the query comes through the scalar cache.
__global__ __launch_bounds__(256) void k_rerank(Dev S, int nq, const float *__restrict__ q, int kc,
                                                const int64_t *__restrict__ cand, int k, int kmul,
                                                const int32_t *__restrict__ kpq, float *__restrict__ dist,
                                                int64_t *__restrict__ labels) {
    const int lane = lane_id();
    const int qi = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6));
    if (qi >= nq) return;
    const int kq = query_k(kpq, k, qi);
    const int nc = min(kq * kmul, kc);
    const int d = S.d, C = S.C;
    uint64_t key = ~0ull;
    if (lane < nc) {
        const int64_t id = cand[(int64_t)qi * kc + lane];
        const uint32_t g = id >= 0 ? S.att[id] : INVALID;
        if (g != INVALID) {
            const f32x4_t *xp = reinterpret_cast<const f32x4_t *>(S.data) + (int64_t)(g / C) * S.dp4 * C + g % C;
            const float *qr = q + (int64_t)qi * d;
            float r = 0.f;
            auto term = [&](float qv, float xv) {
                if (S.metric == 0) {
                    const float t = qv - xv;
                    r = __builtin_fmaf(t, t, r);
                } else {
                    r = __builtin_fmaf(qv, xv, r);
                }
            };
            int c = 0;
            for (; 4 * c + 32 <= d; c += 8) {
                f32x4_t x[8];
#pragma unroll
                for (int i = 0; i < 8; i++) x[i] = xp[(int64_t)(c + i) * C];
#pragma unroll
                for (int i = 0; i < 32; i++) term(qr[4 * c + i], x[i >> 2][i & 3]);
            }
            for (; c < S.dp4; c++) {
                const f32x4_t x = xp[(int64_t)c * C];
#pragma unroll
                for (int i = 0; i < 4; i++)
                    if (4 * c + i < d) term(qr[4 * c + i], x[i]);
            }
            key = make_key(r, (uint32_t)id, S.metric);
        }
    }
    key = wave_sort64(key, true);
    if (lane < k) {
        const int64_t o = (int64_t)qi * k + lane;
        if (lane < kq && key != ~0ull) {
            dist[o] = key_value(key, S.metric);
            labels[o] = (int64_t)(uint32_t)key;
        } else {
            dist[o] = S.metric == 0 ? __int_as_float(0x7F800000) : __int_as_float((int)0xFF800000);
            labels[o] = -1;
        }
    }
}

void launch_rerank(hipStream_t st, const Dev &S, int nq, const float *q, int kc, const int64_t *cand, int k,
                   int kmul, const int32_t *k_per_query, float *dist, int64_t *labels) {
    hipLaunchKernelGGL(k_rerank, dim3((nq + 3) / 4), dim3(256), 0, st, S, nq, q, kc, cand, k, kmul, k_per_query,
                       dist, labels);
}

template <int T, bool WIDE, bool PERS>
static void launch_scan_p(hipStream_t st, const Dev &S, const SearchBufs &W, const float *q, int np_stride,
                          int kcap, int k, const int32_t *kpq, int npairs) {
    const bool sq = (S.d % 4 == 0) && (((uintptr_t)q & 15) == 0);
#define SIVF_LAUNCH_SCAN(KERN, SMEM)                                                                         \
    hipLaunchKernelGGL(KERN, dim3(scan_grid(KERN, S, W, npairs, SMEM)), dim3(64), SMEM, st, S, W.item_list,   \
                       W.item_tile, W.item_chunk, W.list_pairs, q, np_stride, kcap, k, kpq, W.partials, W.gthr)
    if (sq) {
        if (S.metric == 0) SIVF_LAUNCH_SCAN((k_scan_sq<T, 0, WIDE, PERS>), 0);
        else SIVF_LAUNCH_SCAN((k_scan_sq<T, 1, WIDE, PERS>), 0);
        return;
    }
    const size_t smem = (size_t)T * S.dp4 * sizeof(float4);
    if (S.metric == 0) SIVF_LAUNCH_SCAN((k_scan<T, 0, WIDE, PERS>), smem);
    else SIVF_LAUNCH_SCAN((k_scan<T, 1, WIDE, PERS>), smem);
#undef SIVF_LAUNCH_SCAN
}

template <int T, bool WIDE>
static void launch_scan_t(hipStream_t st, const Dev &S, const SearchBufs &W, const float *q, int np_stride,
                          int kcap, int k, const int32_t *kpq, int npairs) {
    if (S.persistent) launch_scan_p<T, WIDE, true>(st, S, W, q, np_stride, kcap, k, kpq, npairs);
    else launch_scan_p<T, WIDE, false>(st, S, W, q, np_stride, kcap, k, kpq, npairs);
}

void launch_search_plan(hipStream_t st, const Dev &S, const SearchBufs &W, int nq, const KClass &cls, int snap,
                        int32_t *heat, int keep_thr) {
    const int np_stride = cls.np_stride;
    const int npairs = nq * np_stride;
    if (keep_thr) nq = 0;   // the kernels below only fill the queries' thresholds with it
    const int T = search_tile(S);
    const int64_t lim = item_limit(S, W, npairs);
    const int xcd_cap = (int)((lim + 7) / 8);
    if (npairs <= SP_PAIRS && S.nlist <= SP_LISTS) {
        hipLaunchKernelGGL(k_inv_small, dim3(1), dim3(1024), (size_t)S.nlist * 12, st, S, T, S.chunk_shift, W.slot_cap,
                           lim, xcd_cap, snap, heat, nq, npairs, W.probes, W.pair_rank, W.list_pairs, W.item_list,
                           W.item_tile, W.item_chunk, cls, W.gthr);
        return;
    }
    const unsigned pb = (unsigned)((npairs + 255) / 256);
    if (S.nlist <= 16384)
        hipLaunchKernelGGL(k_inv_count_lds, dim3((unsigned)((npairs + INV_PB - 1) / INV_PB)), dim3(1024),
                           (size_t)S.nlist * 4, st, S, npairs, W.probes, W.pair_rank, cls, nq, W.gthr);
    else
        hipLaunchKernelGGL(k_inv_count, dim3(pb), dim3(256), 0, st, S, npairs, W.probes, W.pair_rank, cls, nq, W.gthr);
#define SIVF_PLAN(E)                                                                                          \
    hipLaunchKernelGGL(k_inv_plan<E>, dim3(1), dim3(1024), 0, st, S, T, S.chunk_shift, W.slot_cap, lim, xcd_cap, \
                       snap, heat)
    if (S.nlist <= 1024) SIVF_PLAN(1);
    else if (S.nlist <= 4096) SIVF_PLAN(4);
    else if (S.nlist <= 16384) SIVF_PLAN(16);
    else SIVF_PLAN(64);
#undef SIVF_PLAN
    const unsigned ib = (unsigned)((S.nlist + 3) / 4);
    hipLaunchKernelGGL(k_inv_fill, dim3(ib + pb), dim3(256), 0, st, S, T, (int)ib, npairs, W.probes, W.pair_rank,
                       W.list_pairs, W.item_list, W.item_tile, W.item_chunk);
}

bool cert_ok(int storage, int d, int C, int kcap) { return storage == 0 && d <= 256 && C >= 4 && kcap <= 128; }

void launch_search_scan(hipStream_t st, const Dev &S, const SearchBufs &W, int nq, const float *q, int np_stride,
                        int kcap, int k, const int32_t *k_per_query) {
    const int T = search_tile(S);
    const int npairs = nq * np_stride;
    if (T == 16) {   // the schedule setter admits tile 16 only where cert_ok holds
        if (S.metric == 0) launch_scan_cert_l2(st, S, W, q, np_stride, kcap, k, k_per_query, npairs);
        else launch_scan_cert_ip(st, S, W, q, np_stride, kcap, k, k_per_query, npairs);
        return;
    }
    if (kcap > 64) {
        if (T == 2) launch_scan_p<2, true, false>(st, S, W, q, np_stride, kcap, k, k_per_query, npairs);
        else if (T == 8) launch_scan_t<8, true>(st, S, W, q, np_stride, kcap, k, k_per_query, npairs);
        else launch_scan_t<4, true>(st, S, W, q, np_stride, kcap, k, k_per_query, npairs);
    } else {
        if (T == 2) launch_scan_p<2, false, false>(st, S, W, q, np_stride, kcap, k, k_per_query, npairs);
        else if (T == 8) launch_scan_t<8, false>(st, S, W, q, np_stride, kcap, k, k_per_query, npairs);
        else launch_scan_t<4, false>(st, S, W, q, np_stride, kcap, k, k_per_query, npairs);
    }
}

void launch_search_merge(hipStream_t st, const Dev &S, const SearchBufs &W, int nq, const KClass &cls, int kcap,
                         int out_stride, int k, int kmul, const int32_t *k_per_query, float *dist,
                         int64_t *labels, const uint64_t *prior, int prior_stride, uint64_t *keys_out) {
    const int np_stride = cls.np_stride;
    // the MFMA scans publish each query's best k-th key; the VALU scan does not
    uint32_t *gthr = W.gthr;
    // results per query beyond 64 need two keys per lane; four waves per query while 4 nq waves fit the chip
#define SIVF_MERGE(W_, Q_)                                                                                   \
    hipLaunchKernelGGL((k_merge<W_, Q_>), dim3((nq * Q_ + 3) / 4), dim3(256), 0, st, S, nq, np_stride, W.probes,  \
                       W.pair_rank, W.partials, kcap, out_stride, k, kmul, k_per_query, dist, labels, cls, gthr,  \
                       prior, prior_stride, keys_out)
    const bool wide = kmul * k > 64 && out_stride > 64, few = nq <= FILL_ITEMS / 4;
    if (wide && few) SIVF_MERGE(true, 4);
    else if (wide) SIVF_MERGE(true, 1);
    else if (few) SIVF_MERGE(false, 4);
    else SIVF_MERGE(false, 1);
#undef SIVF_MERGE
}

}  // namespace sivf
