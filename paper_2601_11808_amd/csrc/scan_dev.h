// Shared by the scan kernels (search.hip: plan, VALU scans, merge; scan_mfma.hip:
// matrix-core scans): work items, sorted key lists across the lanes of a wave,
// and the launch grids.
#pragma once

#include "sivf_launch.h"

namespace sivf {

__device__ __forceinline__ int cdiv_s(int a, int b) { return (a + b - 1) / b; }

__device__ __forceinline__ int list_chunks(int len, int sh) {
    return len > 0 ? (int)(((int64_t)len + (1ll << sh) - 1) >> sh) : 0;
}

// Work items that fill the chip once: 12 waves on each of 256 CUs.
constexpr int FILL_ITEMS = 3072;

__device__ __forceinline__ uint64_t shfl_xor_u64(uint64_t v, int m) {
    const int lo = __shfl_xor((int)(uint32_t)v, m);
    const int hi = __shfl_xor((int)(uint32_t)(v >> 32), m);
    return ((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo;
}

// ---------------------------------------------------------------- top-k
//
// Per query, the wave keeps its best keys sorted across the lanes (lane i
// holds the i-th best, lanes >= kcap hold ~0).  A key enters only if it beats
// the query's current k-th best (the threshold); such keys are appended to a
// 64-entry LDS buffer with one ballot.  When the buffer is full, and at the
// end of the list, the wave merges it into the sorted list: a bitonic sort of
// the buffer (descending), an element-wise min against the list (the 64
// smallest of both, as a bitonic sequence), and a bitonic merge.

// One compare-exchange step of a bitonic network over the 64 lanes: blocks
// of K lanes, partner distance J; `asc` is the direction of the final order.
template <int K, int J>
__device__ __forceinline__ uint64_t bitonic_step(uint64_t v, bool asc) {
    const int ln = lane_id();
    const uint64_t p = xor_lane_u64<J>(v);
    const bool up = ((ln & K) == 0) == asc;
    const bool keep_min = ((ln & J) == 0) == up;
    const uint64_t lo = p < v ? p : v, hi = p < v ? v : p;
    return keep_min ? lo : hi;
}

// Sort the wave's 64 keys across lanes, ascending or descending.
__device__ __forceinline__ uint64_t wave_sort64(uint64_t v, bool asc) {
    v = bitonic_step<2, 1>(v, asc);
    v = bitonic_step<4, 2>(v, asc);
    v = bitonic_step<4, 1>(v, asc);
    v = bitonic_step<8, 4>(v, asc);
    v = bitonic_step<8, 2>(v, asc);
    v = bitonic_step<8, 1>(v, asc);
    v = bitonic_step<16, 8>(v, asc);
    v = bitonic_step<16, 4>(v, asc);
    v = bitonic_step<16, 2>(v, asc);
    v = bitonic_step<16, 1>(v, asc);
    v = bitonic_step<32, 16>(v, asc);
    v = bitonic_step<32, 8>(v, asc);
    v = bitonic_step<32, 4>(v, asc);
    v = bitonic_step<32, 2>(v, asc);
    v = bitonic_step<32, 1>(v, asc);
    v = bitonic_step<64, 32>(v, asc);
    v = bitonic_step<64, 16>(v, asc);
    v = bitonic_step<64, 8>(v, asc);
    v = bitonic_step<64, 4>(v, asc);
    v = bitonic_step<64, 2>(v, asc);
    v = bitonic_step<64, 1>(v, asc);
    return v;
}

// The 64 smallest keys of a (sorted ascending across lanes) and b (any
// order), sorted ascending: sort b descending; the element-wise min of a and
// b holds the 64 smallest as a bitonic sequence; half-cleaners sort it.
__device__ __forceinline__ uint64_t merge_sorted_with(uint64_t a, uint64_t b) {
    b = wave_sort64(b, false);
    uint64_t c = a < b ? a : b;
    c = bitonic_step<64, 32>(c, true);
    c = bitonic_step<64, 16>(c, true);
    c = bitonic_step<64, 8>(c, true);
    c = bitonic_step<64, 4>(c, true);
    c = bitonic_step<64, 2>(c, true);
    c = bitonic_step<64, 1>(c, true);
    return c;
}

// Half-cleaners: sort a bitonic sequence across the 64 lanes.
__device__ __forceinline__ uint64_t bitonic_clean(uint64_t v, bool asc) {
    v = bitonic_step<64, 32>(v, asc);
    v = bitonic_step<64, 16>(v, asc);
    v = bitonic_step<64, 8>(v, asc);
    v = bitonic_step<64, 4>(v, asc);
    v = bitonic_step<64, 2>(v, asc);
    v = bitonic_step<64, 1>(v, asc);
    return v;
}

// 128-key lists (k > 64): a holds ranks 0..63 and a2 ranks 64..127 (each
// sorted ascending across lanes).  Merge 64 unsorted keys b into them.  With
// b sorted descending, min(a, b) holds the 64 smallest of a and b and
// max(a, b) the rest; none of the former exceeds any key of a2, so the new
// ranks 64..127 are the 64 smallest of max(a, b) and a2.
__device__ __forceinline__ void merge128_with(uint64_t &a, uint64_t &a2, uint64_t b) {
    b = wave_sort64(b, false);
    const uint64_t lo = a < b ? a : b;
    const uint64_t hi = a < b ? b : a;
    a = bitonic_clean(lo, true);
    const uint64_t h = bitonic_clean(hi, false);
    a2 = bitonic_clean(a2 < h ? a2 : h, true);
}

// WIDE: kcap = 128 (two keys per lane).
template <int T, bool WIDE>
struct TopK {
    uint64_t top[T];              // sorted keys, per query (ranks 0..63)
    uint64_t top2[WIDE ? T : 1];  // ranks 64..127
    uint32_t thr[T];              // high word of the query's k-th best key (wave-uniform)
    int cnt[T];                   // keys waiting in the LDS buffer (wave-uniform)
};

// kq: LDS array with each query's k (0 = no results wanted).
template <int T, bool WIDE>
__device__ __forceinline__ void topk_init(TopK<T, WIDE> &K, const int *kq) {
#pragma unroll
    for (int t = 0; t < T; t++) {
        K.top[t] = ~0ull;
        if (WIDE) K.top2[t] = ~0ull;
        K.thr[t] = kq[t] > 0 ? 0xFFFFFFFFu : 0u;
        K.cnt[t] = 0;
    }
}

template <int T, bool WIDE>
__device__ __forceinline__ void topk_flush(TopK<T, WIDE> &K, int t, uint64_t *buf, const int *kq, int kcap) {
    __syncthreads();
    const int ln = lane_id();
    const uint64_t b = ln < K.cnt[t] ? buf[t * 64 + ln] : ~0ull;
    if (WIDE) {
        merge128_with(K.top[t], K.top2[t], b);
        K.top2[t] = ln + 64 < kcap ? K.top2[t] : ~0ull;
        const int r = kq[t] - 1;
        K.thr[t] = (uint32_t)((r < 64 ? readlane_u64(K.top[t], r) : readlane_u64(K.top2[t], r - 64)) >> 32);
    } else {
        uint64_t c = merge_sorted_with(K.top[t], b);
        c = ln < kcap ? c : ~0ull;
        K.top[t] = c;
        K.thr[t] = (uint32_t)(readlane_u64(c, kq[t] - 1) >> 32);
    }
    K.cnt[t] = 0;
    __syncthreads();
}

// Offer one candidate per lane to query t: hi is the high word of its key
// (ordered distance), id its low word.  Keys whose high word is at most the
// threshold's are buffered (a superset of those that beat the k-th key; the
// merge orders them exactly).
template <int T, bool WIDE>
__device__ __forceinline__ void topk_offer(TopK<T, WIDE> &K, int t, bool valid, uint32_t hi, uint32_t id,
                                           uint64_t *buf, const int *kq, int kcap) {
    bool pass = valid && hi <= K.thr[t];
    uint64_t mask = ballot(pass);
    if (mask) {
        int n = __builtin_popcountll(mask);
        if (K.cnt[t] + n > 64) {   // no room: merge first, then re-test against the new threshold
            topk_flush(K, t, buf, kq, kcap);
            pass = valid && hi <= K.thr[t];
            mask = ballot(pass);
            n = __builtin_popcountll(mask);
        }
        if (pass)
            buf[t * 64 + K.cnt[t] + (int)__builtin_popcountll(mask & lanemask_lt())] = ((uint64_t)hi << 32) | id;
        K.cnt[t] += n;
        if (K.cnt[t] == 64) topk_flush(K, t, buf, kq, kcap);
    }
}

// High word of a result key: L2 distances are never negative (the canonical
// sum starts at +0 and adds squares), so their order bits are bits | sign;
// an IP score of -0 ranks as +0.
template <int METRIC>
__device__ __forceinline__ uint32_t key_hi(float v) {
    return METRIC == 0 ? (__float_as_uint(v) | 0x80000000u) : ~ord_bits(zero_sign(v));
}

// Work items are cut into 8 contiguous ranges, one per XCD (blocks are
// dealt to the XCDs round robin): consecutive items share a list, so its
// slabs stay in that XCD's L2.  Two schedules (a template parameter: a loop
// around the scan body costs the hot loop scalar registers):
//  - dispatch (PERS = false): one wave per item; block b takes item b / 8
//    of XCD (b mod 8)'s range; the grid is the host's bound on the item
//    count rounded up to a multiple of 8, and the plan keeps every range
//    within grid / 8 items (surplus waves exit at once);
//  - persistent (PERS = true): a grid of resident waves pulls items from its
//    XCD's counter, then helps the other ranges; every wave ends once all 8
//    counters have passed their range.
#define SIVF_ITEM_LOOP_BEGIN                                                                     \
    for (int xs = 0; xs < (PERS ? 8 : 1); xs++) {                                                \
        const int xx = (int)((blockIdx.x + xs) & 7);                                             \
        const int lo = S.ctl[CTL_XB + xx], hi = S.ctl[CTL_XB + xx + 1];                          \
        for (int it = 0; PERS || it < 1; it++) {                                                 \
            int item;                                                                            \
            if (PERS) {                                                                          \
                item = 0;                                                                        \
                if (threadIdx.x == 0) item = atomicAdd(&S.ctl[CTL_WORK0 + CTL_WORK_STRIDE * xx], 1); \
                item = __builtin_amdgcn_readfirstlane(item) + lo; /* uniform: scalar addressing */ \
            } else {                                                                             \
                item = lo + (int)(blockIdx.x >> 3);                                              \
            }                                                                                    \
            if (item >= hi) break;
#define SIVF_ITEM_LOOP_END \
        }                  \
    }

// Decode a work item: list l, query tile, chunk of positions [p0, p1).
#define SIVF_ITEM_DECODE(TT)                                                                     \
    const int l = item_list[item], tile = item_tile[item];                                       \
    const int nt = min(TT, S.l_qcs[l] - tile * TT);                                              \
    const int len = S.l_snap[l];                                                                 \
    const int p0 = (int)((int64_t)item_chunk[item] << sh);                                       \
    const int p1 = (int)min((int64_t)len, (int64_t)p0 + (1ll << sh));                            \
    const int32_t *pairs = list_pairs + S.l_qoff[l] + tile * TT;

// Partial slot of query t of the item's tile: slot0 + t * nc.  Computed after
// the scan (re-reading the item) so that none of it holds a scalar register
// across the distance loop.
#define SIVF_ITEM_SLOT(TT)                                                                       \
    const int nc = list_chunks(len, S.ctl[CTL_CHUNK]);                                           \
    const int64_t slot0 = (int64_t)S.l_pbase[l] + (int64_t)tile * TT * nc + item_chunk[item];

__device__ __forceinline__ int query_k(const int32_t *kpq, int k, int qi) {
    int kq = kpq ? kpq[qi] : k;
    return kq < 0 ? 0 : (kq > k ? k : kq);
}

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

template <int DT>
__device__ __forceinline__ f32x4_t mfma_16x16x32(uint4 a, uint4 b, f32x4_t c) {
    if constexpr (DT == 1)
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b),
                                                      c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8_t, a), __builtin_bit_cast(f16x8_t, b),
                                                     c, 0, 0, 0);
}

constexpr int MQ = 16;       // queries per MFMA tile
constexpr int MKB = 8;       // k-blocks of 32 dims: d <= 256
constexpr int MBUF = 96;     // candidate buffer per query (a step adds at most 64)


// Work items of a call without splitting: tiles of T pairs per list.  The
// plan may split long lists until the items reach twice this, or twice what
// fills the chip (or the buffer); the dispatch grid covers that bound.
static inline int64_t items_unsplit(const Dev &S, int npairs) {
    const int T = search_tile(S);
    return (npairs + T - 1) / T + (npairs < S.nlist ? npairs : S.nlist);
}

static inline int64_t item_limit(const Dev &S, const SearchBufs &W, int npairs) {
    int64_t lim = 2 * items_unsplit(S, npairs);
    lim = lim > 2 * FILL_ITEMS ? lim : 2 * FILL_ITEMS;   // room to split the lists of a small batch
    return lim < W.item_cap ? lim : W.item_cap;
}

// Grid of a scan launch: the call's item bound rounded up to a multiple of 8
// (dispatch), or the waves that fit on the chip at the kernel's occupancy
// (persistent).
template <typename K>
static unsigned scan_grid(K kernel, const Dev &S, const SearchBufs &W, int npairs, size_t smem) {
    if (!S.persistent) {
        const int64_t g = (item_limit(S, W, npairs) + 7) / 8 * 8;
        return (unsigned)(g < 8 ? 8 : g);
    }
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, 64, smem) != hipSuccess || per_cu < 1)
        per_cu = 8;
    static int cus = 0;   // compute units of the first device used (all GPUs of a node are one part)
    if (cus == 0) {
        int dev = 0, n = 0;
        cus = (hipGetDevice(&dev) == hipSuccess &&
               hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && n > 0)
                  ? n
                  : 256;
    }
    return (unsigned)(per_cu * cus);
}

}  // namespace sivf
