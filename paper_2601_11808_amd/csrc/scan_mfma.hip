// Matrix-core scans of the slab-resident lists: the reduced-precision scan
// (bf16 / fp16 slabs) and the certified FP32 scan.  Work items, partial lists and
// schedules as in search.hip.
#include "scan_dev.h"

namespace sivf {

// ------------------------------------------------ reduced-precision scan
//
// Slabs in bf16 / fp16 ([slab][8-dim chunk][slot], 16 bytes per slot and
// chunk).  One wave scans a list for a tile of 16 queries with
// v_mfma_f32_16x16x32_{bf16,f16}: the A operand is 16 slots x 32 dims (lane l:
// slot l % 16, dims 8 (l / 16) .. +8 of the k-block), B the 16 queries
// rounded the same way, C the 16 x 16 fp32 scores (lane l: slots
// 4 (l / 16) .. +4, query l % 16).  Approximate distances:
// |x~|^2 + |q~|^2 - 2 x~.q~ (L2) or x~.q~ (IP), with FP32 accumulation.  Each
// query keeps its best kmul * k approximate candidates; the exact FP32
// re-rank over the shadow rows (k_rerank) decides the final order.

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

// Merge query t's buffered candidates into its sorted list (lane i = i-th
// best) and return the list's kq-th key's high word.
template <int NQ>
__device__ __forceinline__ uint32_t mfma_flush(uint64_t (&top)[NQ], int t, const uint64_t *buf, int cnt, int kq,
                                               int kcap) {
    const int lane = lane_id();
    const uint64_t b0 = lane < cnt ? buf[t * MBUF + lane] : ~0ull;
    uint64_t c = merge_sorted_with(top[t], b0);
    if (cnt > 64) {
        const uint64_t b1 = lane + 64 < cnt ? buf[t * MBUF + 64 + lane] : ~0ull;
        c = merge_sorted_with(c, b1);
    }
    c = lane < kcap ? c : ~0ull;
    top[t] = c;
    return kq > 0 ? (uint32_t)(readlane_u64(c, kq - 1) >> 32) : 0u;
}

template <int METRIC, int DT, int NKB, bool PERS>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(3, 8))) void k_scan_mfma(Dev S, const int32_t *__restrict__ item_list,
                                                  const int32_t *__restrict__ item_tile,
                                                  const int32_t *__restrict__ item_chunk,
                                                  const int32_t *__restrict__ list_pairs,
                                                  const float *__restrict__ q, int np_stride, int kcap, int k,
                                                  int kmul, const int32_t *__restrict__ kpq,
                                                  uint64_t *__restrict__ partials, uint32_t *__restrict__ gthr) {
    __shared__ uint64_t buf[MQ * MBUF];
    __shared__ int scnt[MQ], skq[MQ];
    const int lane = threadIdx.x, qcol = lane & 15, kgrp = lane >> 4;
    const int d = S.d, C = S.C, dp8 = S.dp8, sh = S.ctl[CTL_CHUNK];
    const int cs = __builtin_ctz(C), cm = C - 1;   // slab capacities are powers of two
    SIVF_ITEM_LOOP_BEGIN
    SIVF_ITEM_DECODE(MQ)
    __syncthreads();
    if (lane < MQ) {
        skq[lane] = lane < nt ? min(kmul * query_k(kpq, k, pairs[lane] / np_stride), kcap) : 0;
        scnt[lane] = 0;
    }
    // B operand: query qcol, dims 32 kb + 8 kgrp .. +8, rounded like the slabs
    const int qg = pairs[qcol < nt ? qcol : 0] / np_stride;   // query of column qcol
    const float *qr = q + (int64_t)qg * d;
    uint4 bq[NKB];
    float qn = 0.f;
#pragma unroll
    for (int kb = 0; kb < NKB; kb++) {
        uint32_t h[8];
#pragma unroll
        for (int e = 0; e < 8; e++) {
            const int j = 32 * kb + 8 * kgrp + e;
            const float v = j < d ? qr[j] : 0.f;
            h[e] = DT == 1 ? to_bf16_bits(v) : to_f16_bits(v);
            const float r = DT == 1 ? bf16_bits_to_float(h[e]) : f16_bits_to_float(h[e]);
            qn = fmaf(r, r, qn);
        }
        bq[kb] = make_uint4(h[0] | (h[1] << 16), h[2] | (h[3] << 16), h[4] | (h[5] << 16), h[6] | (h[7] << 16));
    }
    qn += __shfl_xor(qn, 16);
    qn += __shfl_xor(qn, 32);
    __syncthreads();
    uint32_t thr = skq[qcol] > 0 ? 0xFFFFFFFFu : 0u;   // threshold of query qcol (high word of its k-th key)
    // The same threshold as a float: a value passes when its key's high word is
    // at most thr, i.e. (L2) !(v > thr_f) or (IP) !(v < thr_f).  thr = ~0
    // (list not yet full) maps to NaN, which passes everything.
    const bool live = qcol < nt && skq[qcol] > 0;
    float thr_f = METRIC == 0 ? from_ord(thr) : from_ord(~thr);
    uint64_t top[MQ];
#pragma unroll
    for (int t = 0; t < MQ; t++) top[t] = ~0ull;

    const int nslab = (len + cm) >> cs;
    int wbase = -(1 << 30), wslab = 0;
    const bool one_slab = cs >= 6 && !(p0 & 63);   // steps never straddle slabs
    for (int base = p0; base < p1; base += 64) {
        const int last_ord = min(base + 63, p1 - 1) >> cs;
        if (last_ord >= wbase + 64) {
            wbase = base >> cs;
            wslab = (wbase + lane < nslab) ? slab_of(S, l, wbase + lane) : 0;
        }
        // the 4 result rows of this lane in row group rg are positions
        // base + 16 rg + 4 kgrp .. +3: one slab (C >= 4), 16-byte aligned slots.
        // A operands of row group rg: slot 16 rg + qcol, 8-dim chunks 4 kb + kgrp;
        // two row groups in flight.  Chunks past the row repeat its last chunk
        // (their B lanes are zero); positions past the item read its last row
        // and are masked below.
        int64_t g4[4];
        const uint4 *hr[4];
        if (one_slab) {
            // the step's 64 positions lie in one slab: a scalar slab index
            const int64_t sb = __builtin_amdgcn_readlane(wslab, (base >> cs) - wbase);
#pragma unroll
            for (int rg = 0; rg < 4; rg++) {
                const int p = base + 16 * rg + 4 * kgrp, pr = base + 16 * rg + qcol;
                g4[rg] = sb * C + ((p < p1 ? p : ((p1 - 1) & ~3)) & cm);
                hr[rg] = S.hdata + sb * dp8 * C + ((pr < p1 ? pr : p1 - 1) & cm);
            }
        } else {
#pragma unroll
            for (int rg = 0; rg < 4; rg++) {
                const int p = base + 16 * rg + 4 * kgrp;
                const int pc = p < p1 ? p : ((p1 - 1) & ~3);
                g4[rg] = (int64_t)__shfl(wslab, (pc >> cs) - wbase) * C + (pc & cm);
            }
#pragma unroll
            for (int rg = 0; rg < 4; rg++) {
                const int p = base + 16 * rg + qcol;
                const int pc = p < p1 ? p : p1 - 1;
                const int slab = __shfl(wslab, (pc >> cs) - wbase);
                hr[rg] = S.hdata + (int64_t)slab * dp8 * C + (pc & cm);
            }
        }
        // the best R k-th key any work item has published for this query: a candidate behind it cannot
        // enter the query's final list (those R k keys are real candidates), so it tightens the filter
        const uint32_t pub = live ? __hip_atomic_load(gthr + qg, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : ~0u;
        float4 xn4[4] = {};
        if (METRIC == 0) {
#pragma unroll
            for (int rg = 0; rg < 4; rg++) xn4[rg] = *reinterpret_cast<const float4 *>(S.xnorm + g4[rg]);
        }
        f32x4_t acc[4];
        uint4 a0[NKB], a1[NKB];
        auto load_a = [&](uint4 (&a)[NKB], const uint4 *h) {
#pragma unroll
            for (int kb = 0; kb < NKB; kb++) a[kb] = h[(int64_t)min(4 * kb + kgrp, dp8 - 1) * C];
        };
        auto mma = [&](const uint4 (&a)[NKB]) {
            f32x4_t c = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kb = 0; kb < NKB; kb++) c = mfma_16x16x32<DT>(a[kb], bq[kb], c);
            return c;
        };
        load_a(a0, hr[0]);
        load_a(a1, hr[1]);
        acc[0] = mma(a0);
        load_a(a0, hr[2]);
        acc[1] = mma(a1);
        load_a(a1, hr[3]);
        acc[2] = mma(a0);
        acc[3] = mma(a1);
        if (pub < thr) {
            thr = pub;
            thr_f = METRIC == 0 ? from_ord(thr) : from_ord(~thr);
        }
        float vv[16];
        uint32_t pmask = 0;
#pragma unroll
        for (int rg = 0; rg < 4; rg++) {
            const float xs[4] = {xn4[rg].x, xn4[rg].y, xn4[rg].z, xn4[rg].w};
#pragma unroll
            for (int j = 0; j < 4; j++) {
                const float v = METRIC == 0 ? fmaf(-2.f, acc[rg][j], qn + xs[j]) : acc[rg][j];
                vv[4 * rg + j] = v;
                const bool pass = METRIC == 0 ? !(v > thr_f) : !(v < thr_f);
                pmask |= (pass ? 1u : 0u) << (4 * rg + j);
            }
        }
        if (!live) pmask = 0;
        // in range and (lazy deletes) live
        pmask &= lane_valid16(step_valid(S, base, p1, wslab, wbase, cs, cm), kgrp);
        if (ballot(pmask != 0)) {
            // offsets of this lane's candidates among the 4 lanes of its query
            const int np = __builtin_popcount(pmask);
            int incl = np;
            int u = __shfl_up(incl, 16);
            if (kgrp >= 1) incl += u;
            u = __shfl_up(incl, 32);
            if (kgrp >= 2) incl += u;
            int at = scnt[qcol] + incl - np;
#pragma unroll
            for (int rg = 0; rg < 4; rg++) {
                if ((pmask >> (4 * rg)) & 0xFu) {
                    const uint4 id4 = *reinterpret_cast<const uint4 *>(S.sids + g4[rg]);
                    const uint32_t ids[4] = {id4.x, id4.y, id4.z, id4.w};
#pragma unroll
                    for (int j = 0; j < 4; j++) {
                        if ((pmask >> (4 * rg + j)) & 1u) {
                            const float v = vv[4 * rg + j];
                            const uint32_t hi = METRIC == 0 ? ord_bits(v) : ~ord_bits(zero_sign(v));
                            buf[qcol * MBUF + at] = ((uint64_t)hi << 32) | ids[j];
                            at++;
                        }
                    }
                }
            }
            __syncthreads();
            if (kgrp == 3) scnt[qcol] = at;   // the last lane of the query holds the new count
            __syncthreads();
            // merge buffers that could overflow on the next step, and fill a
            // query's list as soon as it has k candidates (sets its threshold)
            bool need = false;
            if (lane < MQ) {
                const int cnt = scnt[lane];
                need = cnt > MBUF - 64 || (thr == 0xFFFFFFFFu && cnt > 0 && cnt >= skq[lane]);
            }
            const uint64_t fm = ballot(need);
            if (fm) {
#pragma unroll
                for (int t = 0; t < MQ; t++) {
                    if ((fm >> t) & 1ull) {
                        const uint32_t nthr = mfma_flush<MQ>(top, t, buf, scnt[t], skq[t], kcap);
                        // publish a full list's R k-th key for the query's other work items (the query
                        // index is read while the whole wave is active)
                        const int qt = __builtin_amdgcn_readlane(qg, t);
                        if (lane == 0 && nthr != 0xFFFFFFFFu)
                            __hip_atomic_fetch_min(gthr + qt, nthr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        if (qcol == t) {
                            thr = nthr;
                            thr_f = METRIC == 0 ? from_ord(thr) : from_ord(~thr);
                        }
                    }
                }
                __syncthreads();
                if (lane < MQ && ((fm >> lane) & 1ull)) scnt[lane] = 0;
                __syncthreads();
            }
        }
    }
    SIVF_ITEM_SLOT(MQ)
#pragma unroll
    for (int t = 0; t < MQ; t++) {
        if (t < nt) {
            const int cnt = scnt[t];
            if (cnt > 0) mfma_flush<MQ>(top, t, buf, cnt, skq[t], kcap);
            if (lane < kcap) partials[(slot0 + (int64_t)t * nc) * kcap + lane] = top[t];
        }
    }
    SIVF_ITEM_LOOP_END
}

// Insert key c into a list sorted ascending across lanes s0 .. s0 + KC - 1
// (lane s0 + i holds the i-th smallest); the largest key drops out and the
// other lanes keep their keys.  Keys are distinct.
template <int KC>
__device__ __forceinline__ uint64_t sorted_insert(uint64_t a, uint64_t c, int s0) {
    const int lane = lane_id();
    // previous lane's key: DPP wave_shr:1 (lane 0 keeps its own, unused)
    const uint32_t plo = (uint32_t)__builtin_amdgcn_update_dpp((int)(uint32_t)a, (int)(uint32_t)a, 0x138, 0xf, 0xf, false);
    const uint32_t phi = (uint32_t)__builtin_amdgcn_update_dpp((int)(uint32_t)(a >> 32), (int)(uint32_t)(a >> 32), 0x138,
                                                                0xf, 0xf, false);
    const uint64_t prev = ((uint64_t)phi << 32) | plo;
    const uint64_t r = a < c ? a : ((lane == s0 || prev < c) ? c : prev);
    return (KC == 64 || (lane >= s0 && lane < s0 + KC)) ? r : a;
}

// Canonical FP32 value of one (row, query) pair, exactly as the VALU scan
// computes it (one fma per dimension, ascending, over the padded chunks);
// four chunks of loads in flight.  qv4: the query's zero-padded row in LDS.
template <int METRIC>
__device__ __forceinline__ void cert_chunk(float &r, float4 qv, float4 xv) {
    if (METRIC == 0) {
        float e;
        e = qv.x - xv.x;
        r = __builtin_fmaf(e, e, r);
        e = qv.y - xv.y;
        r = __builtin_fmaf(e, e, r);
        e = qv.z - xv.z;
        r = __builtin_fmaf(e, e, r);
        e = qv.w - xv.w;
        r = __builtin_fmaf(e, e, r);
    } else {
        r = __builtin_fmaf(qv.x, xv.x, r);
        r = __builtin_fmaf(qv.y, xv.y, r);
        r = __builtin_fmaf(qv.z, xv.z, r);
        r = __builtin_fmaf(qv.w, xv.w, r);
    }
}

template <int METRIC>
__device__ __forceinline__ float cert_exact(const float4 *__restrict__ xp, int C, int dp4, const float4 *qv4) {
    float r = 0.f;
    int c0 = 0;
    for (; c0 + 4 <= dp4; c0 += 4) {
        float4 xv[4];
#pragma unroll
        for (int u = 0; u < 4; u++) xv[u] = xp[(int64_t)(c0 + u) * C];
#pragma unroll
        for (int u = 0; u < 4; u++) cert_chunk<METRIC>(r, qv4[c0 + u], xv[u]);
    }
    for (; c0 < dp4; c0++) cert_chunk<METRIC>(r, qv4[c0], xp[(int64_t)c0 * C]);
    return r;
}

template <int NB>
__device__ __forceinline__ void cert_load_a(float4 (&a)[NB], const float4 *__restrict__ xr, int C, int kgrp, int dp4) {
#pragma unroll
    for (int b = 0; b < NB; b++) a[b] = xr[(int64_t)min(4 * b + kgrp, dp4 - 1) * C];
}

// 16 slots x 16 queries over all dimensions; B operand (query l % 16, chunk
// 4 b + l / 16) read from the LDS query rows.
template <int NB>
__device__ __forceinline__ f32x4_t cert_mfma(const float4 (&a)[NB], const float4 *qrow, int kgrp, int dp4) {
    f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
    // the next chunk's LDS read is in flight during this chunk's MFMAs
    float4 nb = kgrp < dp4 ? qrow[kgrp] : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int b = 0; b < NB; b++) {
        const float4 bv = nb;
        if (b + 1 < NB) {
            const int c = 4 * b + 4 + kgrp;
            nb = c < dp4 ? qrow[c] : make_float4(0.f, 0.f, 0.f, 0.f);
        }
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[b].x, bv.x, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[b].y, bv.y, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[b].z, bv.z, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[b].w, bv.w, acc, 0, 0, 0);
    }
    return acc;
}

// ------------------------------------------------ certified FP32 MFMA scan
//
// FP32 slabs with results identical to the canonical scan.  For this contraction
// v_mfma_f32_16x16x4_f32 does four times the work per cycle of the sub + fma VALU
// form; it gives approximate values for 16 slots x 16 queries:
// Dt = |x|^2 + |q|^2 - 2 x.q (L2) or -x.q (IP, as a distance).  A slot can be
// among a query's k best only if Dt - e is at most the query's current k-th best
// canonical value; only those pairs get their canonical FP32 distance recomputed
// (sequential fma over ascending dimensions, exactly as the VALU scan computes it)
// and inserted into the query's exact sorted list.
//
// Half-width e.  With rounding error at most one unit 2^-24 per operation, the MFMA
// form (norms included) differs from the exact value by at most (2d + 4) 2^-24
// (|x| + |q|)^2 and the canonical sum by (d + 2) 2^-24 |q - x|^2; IP: 2d and d times
// 2^-24 |x||q|.  The kernel uses cf (|x| + |q|)^2 with cf = (5d + 32) 2^-24 (IP:
// (4d + 32) 2^-24 |x||q|), plus 2^-122 sqrt(d) (|x| + |q|) + 2^-120 d for underflow,
// relaxed to e = e1 (|x|^2 + |q|^2) + e0 so that no square root is needed (the
// margin covers the rounding of the fp32 norms and of e).  An overflowing value gives
// inf or NaN in the test, and both pass.
//
// Before a query has k exact values (the first step of a work item), its threshold
// is the k-th smallest upper bound Dt + e among the step's candidates, found by
// bisection: at least k candidates lie at or below it, so the k best do too.
//
// Layout.  A operand (lane l): slot l % 16 of the row group, the 4 dimensions of
// chunk 4 b + l / 16 (one float4), fed to 4 consecutive MFMAs one component each;
// the B operand holds the same dimensions of query l % 16 (read from the tile's
// query rows in LDS), so every MFMA pairs equal dimensions and the 4 x NB MFMAs of
// a row group cover all 16 NB dimensions.  C (lane l): slots 4 (l / 16) .. +3,
// query l % 16.  Passing pairs are queued in LDS and recomputed one per lane,
// in full rounds of 64 (the queue drains early when a query has no k-th value
// yet, before the slab window moves, and at the end of the item).
// Exact lists: KC keys per query sorted across KC lanes, 64 / KC queries per
// register (KC = 16 for kcap 16, else 64).  KC = 128 (k up to 128): ranks
// 0..63 stay in registers as for KC = 64; ranks 64..127 are kept only for
// queries whose k exceeds 64, in the upper half of the query's own partial
// slot (read and written back by the inserting lanes, each its own rank; an
// LDS copy would cost the kernel a third of its resident waves); a key that
// enters the low half pushes its largest key down into the high half.
template <int METRIC, int NB, bool PERS, int KC>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(3, 8))) void k_scan_cert(Dev S, const int32_t *__restrict__ item_list,
                                                  const int32_t *__restrict__ item_tile,
                                                  const int32_t *__restrict__ item_chunk,
                                                  const int32_t *__restrict__ list_pairs,
                                                  const float *__restrict__ q, int np_stride, int kcap, int k,
                                                  const int32_t *__restrict__ kpq,
                                                  uint64_t *__restrict__ partials, uint32_t *__restrict__ gthr) {
    extern __shared__ float4 sqr[];    // the tile's 16 query rows, zero-padded to dp4 chunks, stride dp4 + 1
    __shared__ uint32_t pq[64 * MQ + 64];   // queued passing pairs: window position << 4 | query
    __shared__ int skq[MQ];
    const int lane = threadIdx.x, qcol = lane & 15, kgrp = lane >> 4;
    const int d = S.d, C = S.C, dp4 = S.dp4, sh = S.ctl[CTL_CHUNK];
    const int qs = dp4 + 1;   // LDS row stride: rows start in different banks
    const int cs = __builtin_ctz(C), cm = C - 1;   // slab capacities are powers of two
    // half-width e = e1 (|x|^2 + |q|^2) + e0, from (|x| + |q|)^2 <= 2 (|x|^2 + |q|^2),
    // |x||q| <= (|x|^2 + |q|^2) / 2 and |x| + |q| <= 1 + (|x|^2 + |q|^2)
    const float cf = METRIC == 0 ? (5.0f * d + 32.0f) * 0x1p-24f : (4.0f * d + 32.0f) * 0x1p-24f;
    const float ca = sqrtf((float)d) * 0x1p-122f, cb = (float)d * 0x1p-120f;
    const float e1 = (METRIC == 0 ? 2.f * cf : 0.5f * cf) + ca, e0 = ca + cb;
    SIVF_ITEM_LOOP_BEGIN
    SIVF_ITEM_DECODE(MQ)
    __syncthreads();
    if (lane < MQ) {
        const int qi = pairs[lane < nt ? lane : 0] / np_stride;
        skq[lane] = lane < nt ? min(query_k(kpq, k, qi), kcap) : 0;
    }
    for (int i = lane; i < MQ * dp4; i += 64) {
        const int t = i / dp4, j = 4 * (i - t * dp4);
        const float *qr = q + (int64_t)(pairs[t < nt ? t : 0] / np_stride) * d;
        float4 v;
        v.x = j < d ? qr[j] : 0.f;
        v.y = j + 1 < d ? qr[j + 1] : 0.f;
        v.z = j + 2 < d ? qr[j + 2] : 0.f;
        v.w = j + 3 < d ? qr[j + 3] : 0.f;
        sqr[t * qs + (j >> 2)] = v;
    }
    __syncthreads();
    const int qg = pairs[qcol < nt ? qcol : 0] / np_stride;   // query of column qcol
    float qn2 = 0.f;   // |q|^2 of query qcol
#pragma unroll
    for (int b = 0; b < NB; b++) {
        const int c = 4 * b + kgrp;
        const float4 v = c < dp4 ? sqr[qcol * qs + c] : make_float4(0.f, 0.f, 0.f, 0.f);
        qn2 = fmaf(v.x, v.x, qn2);
        qn2 = fmaf(v.y, v.y, qn2);
        qn2 = fmaf(v.z, v.z, qn2);
        qn2 = fmaf(v.w, v.w, qn2);
    }
    qn2 += __shfl_xor(qn2, 16);
    qn2 += __shfl_xor(qn2, 32);
    __syncthreads();
    uint32_t thr = skq[qcol] > 0 ? 0xFFFFFFFFu : 0u;   // high word of query qcol's k-th exact key
    // the k-th exact value as a float (L2: distance, IP: score); ~0 maps to NaN, which passes all
    const bool live = qcol < nt && skq[qcol] > 0;
    float thr_f = METRIC == 0 ? from_ord(thr) : from_ord(~thr);
    // sorted exact lists: query t in register t / QPR, lanes KC (t % QPR) .. +KC-1
    // (KC = 128: ranks 0..63 in register t, the rest in LDS)
    constexpr int QPR = KC == 128 ? 1 : 64 / KC, NR = MQ / QPR;
    uint64_t top[NR];
#pragma unroll
    for (int r = 0; r < NR; r++) top[r] = ~0ull;
    uint32_t hset = 0;   // KC = 128: queries whose ranks 64..127 have been written to their slot

    const int nslab = (len + cm) >> cs;
    int wbase = -(1 << 30), wslab = 0;
    int qn = 0;   // queued pairs (fewer than 64 carry over to the next step)
    const bool one_slab = cs >= 6 && !(p0 & 63);   // steps never straddle slabs
    for (int base = p0; base < p1; base += 64) {
        const int last_ord = min(base + 63, p1 - 1) >> cs;
        if (last_ord >= wbase + 64) {
            wbase = base >> cs;
            wslab = (wbase + lane < nslab) ? slab_of(S, l, wbase + lane) : 0;
        }
        // the 4 result rows of this lane in row group rg: positions base + 16 rg + 4 kgrp .. +3
        // A operands of row group rg: slot 16 rg + qcol, chunks 4 b + kgrp; two
        // row groups in flight (the loads of the next overlap this one's MFMAs).
        // Chunks past the row repeat its last chunk (their B lanes are zero and
        // stored values are finite); positions past the item read its last row
        // and are masked below.
        int64_t g4[4];
        const float4 *xr[4];
        if (one_slab) {
            // the step's 64 positions lie in one slab: a scalar slab index
            const int64_t sb = __builtin_amdgcn_readlane(wslab, (base >> cs) - wbase);
#pragma unroll
            for (int rg = 0; rg < 4; rg++) {
                const int p = base + 16 * rg + 4 * kgrp, pr = base + 16 * rg + qcol;
                g4[rg] = sb * C + ((p < p1 ? p : ((p1 - 1) & ~3)) & cm);
                xr[rg] = S.data + sb * dp4 * C + ((pr < p1 ? pr : p1 - 1) & cm);
            }
        } else {
#pragma unroll
            for (int rg = 0; rg < 4; rg++) {
                const int p = base + 16 * rg + 4 * kgrp;
                const int pc = p < p1 ? p : ((p1 - 1) & ~3);
                g4[rg] = (int64_t)__shfl(wslab, (pc >> cs) - wbase) * C + (pc & cm);
            }
#pragma unroll
            for (int rg = 0; rg < 4; rg++) {
                const int p = base + 16 * rg + qcol;
                const int pc = p < p1 ? p : p1 - 1;
                const int slab = __shfl(wslab, (pc >> cs) - wbase);
                xr[rg] = S.data + (int64_t)slab * dp4 * C + (pc & cm);
            }
        }
        // the best k-th key value any work item has published for this query: a pair behind it cannot
        // enter the query's final k (those k keys are real candidates), so it serves as the threshold
        const uint32_t pub = live ? __hip_atomic_load(gthr + qg, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : ~0u;
        float4 xn4[4];
#pragma unroll
        for (int rg = 0; rg < 4; rg++) xn4[rg] = *reinterpret_cast<const float4 *>(S.xnorm + g4[rg]);
        f32x4_t acc[4];
        float4 a0[NB], a1[NB];
        cert_load_a<NB>(a0, xr[0], C, kgrp, dp4);
        cert_load_a<NB>(a1, xr[1], C, kgrp, dp4);
        acc[0] = cert_mfma<NB>(a0, sqr + qcol * qs, kgrp, dp4);
        cert_load_a<NB>(a0, xr[2], C, kgrp, dp4);
        acc[1] = cert_mfma<NB>(a1, sqr + qcol * qs, kgrp, dp4);
        cert_load_a<NB>(a1, xr[3], C, kgrp, dp4);
        acc[2] = cert_mfma<NB>(a0, sqr + qcol * qs, kgrp, dp4);
        acc[3] = cert_mfma<NB>(a1, sqr + qcol * qs, kgrp, dp4);
        // distance space (L2: the distance; IP: minus the score): value v and
        // certified half-width e of every (slot, query) pair of this lane
        float vv[16], ee[16];
        // bit 4 rg + j: position 16 rg + 4 kgrp + j in range and (lazy deletes) live
        const uint32_t vm = lane_valid16(step_valid(S, base, p1, wslab, wbase, cs, cm), kgrp);
#pragma unroll
        for (int rg = 0; rg < 4; rg++) {
            const float xs[4] = {xn4[rg].x, xn4[rg].y, xn4[rg].z, xn4[rg].w};
#pragma unroll
            for (int j = 0; j < 4; j++) {
                const float sq = qn2 + xs[j];
                vv[4 * rg + j] = METRIC == 0 ? fmaf(-2.f, acc[rg][j], sq) : -acc[rg][j];
                ee[4 * rg + j] = fmaf(e1, sq, e0);
            }
        }
        if (pub < thr) {
            thr = pub;
            thr_f = METRIC == 0 ? from_ord(thr) : from_ord(~thr);
        }
        // the query's k-th best value so far in distance space (NaN: none yet, all pass)
        float thd = METRIC == 0 ? thr_f : -thr_f;
        const bool warm = live && thr == 0xFFFFFFFFu;
        if (ballot(warm)) {
            // No k-th value yet: bound it by the k-th smallest upper bound v + e
            // among this step's candidates of the query (lanes qcol + 16 i hold
            // them): at least k candidates lie at or below it, so the k best
            // do too.  Bisection keeps count(v + e <= hi) >= k.
            int nv = 0;
            float mn = __int_as_float(0x7F800000), mx = -__int_as_float(0x7F800000);
#pragma unroll
            for (int i = 0; i < 16; i++) {
                float u = vv[i] + ee[i];
                if (!(u <= __int_as_float(0x7F800000))) u = __int_as_float(0x7F800000);   // NaN: +inf
                if ((vm >> i) & 1u) {
                    nv++;
                    mn = fminf(mn, u);
                    mx = fmaxf(mx, u);
                }
            }
            nv += __shfl_xor(nv, 16);
            nv += __shfl_xor(nv, 32);
            mn = fminf(mn, __shfl_xor(mn, 16));
            mn = fminf(mn, __shfl_xor(mn, 32));
            mx = fmaxf(mx, __shfl_xor(mx, 16));
            mx = fmaxf(mx, __shfl_xor(mx, 32));
            const int kq = skq[qcol];
            float lo = mn, hi = mx;
            for (int it = 0; it < 10; it++) {
                const float mid = lo + 0.5f * (hi - lo);
                int c = 0;
#pragma unroll
                for (int i = 0; i < 16; i++) {
                    const float u = vv[i] + ee[i];
                    c += (((vm >> i) & 1u) && u <= mid) ? 1 : 0;
                }
                c += __shfl_xor(c, 16);
                c += __shfl_xor(c, 32);
                if (c >= kq) hi = mid;
                else lo = mid;
            }
            if (warm && nv >= kq) thd = hi;
        }
        uint32_t pmask = 0;
#pragma unroll
        for (int i = 0; i < 16; i++) pmask |= (!(vv[i] - ee[i] > thd) ? 1u : 0u) << i;
        if (!live) pmask = 0;
        pmask &= vm;
        if (ballot(pmask != 0)) {
            // queue the passing (position, query) pairs in lane order
            const int np = __builtin_popcount(pmask);
            const int incl = wave_incl_scan_dpp(np);
            int at = qn + incl - np;
            qn += __builtin_amdgcn_readlane(incl, 63);
            const int wpos = base - (wbase << cs);   // queued positions are relative to the slab window
            uint32_t m = pmask;
            while (m) {
                const int bit = __builtin_ctz(m);
                m &= m - 1;
                pq[at++] = ((uint32_t)(wpos + 16 * (bit >> 2) + 4 * kgrp + (bit & 3)) << 4) | (uint32_t)qcol;
            }
        }
        // Recompute full rounds of 64 pairs; everything when a query still waits
        // for its first k-th value, before the slab window moves, and at the end.
        const int nb = base + 64;
        const bool drain = ballot(live && thr == 0xFFFFFFFFu) != 0 || nb >= p1 ||
                           (min(nb + 63, p1 - 1) >> cs) >= wbase + 64;
        const int nproc = drain ? qn : (qn & ~63);
        if (nproc > 0) {
            __syncthreads();
            for (int r0 = 0; r0 < nproc; r0 += 64) {
                const bool act = r0 + lane < nproc;
                const uint32_t e = pq[act ? r0 + lane : r0];
                const int t = (int)(e & 15), pw = (int)(e >> 4);
                const int slab = __shfl(wslab, pw >> cs), slot = pw & cm;
                uint64_t key = ~0ull;
                if (act) {
                    const float r = cert_exact<METRIC>(S.data + (int64_t)slab * dp4 * C + slot, C, dp4, sqr + t * qs);
                    key = ((uint64_t)key_hi<METRIC>(r) << 32) | S.sids[(int64_t)slab * C + slot];
                }
                // insert the exact keys into their queries' sorted lists, one at a time
#pragma unroll
                for (int t2 = 0; t2 < MQ; t2++) {
                    uint64_t bm = ballot(act && t == t2);
                    if (bm) {
                        const int kq = __builtin_amdgcn_readfirstlane(skq[t2]);   // > 0: only live queries have pairs
                        uint64_t hi = ~0ull;      // KC = 128, k > 64: ranks 64..127
                        uint64_t *hdst = nullptr;
                        if constexpr (KC == 128) {
                            if (kq > 64) {
                                SIVF_ITEM_SLOT(MQ)
                                hdst = partials + (slot0 + (int64_t)t2 * nc) * kcap + 64;
                                if ((hset >> t2) & 1u) hi = hdst[lane];
                                hset |= 1u << t2;
                            }
                        }
                        // only keys below the query's current k-th key can change its k best
                        uint64_t kth;
                        if constexpr (KC == 128) kth = kq <= 64 ? readlane_u64(top[t2], kq - 1) : readlane_u64(hi, kq - 65);
                        else kth = readlane_u64(top[t2 / QPR], KC * (t2 % QPR) + kq - 1);
                        bm = ballot(act && t == t2 && key < kth);
                        while (bm) {
                            const int src = (int)__builtin_ctzll(bm);
                            bm &= bm - 1;
                            uint64_t c = readlane_u64(key, src);
                            if constexpr (KC == 128) {
                                // a key below the low half's largest enters it and pushes that one down
                                const uint64_t lmax = readlane_u64(top[t2], 63);
                                if (c < lmax) {
                                    top[t2] = sorted_insert<64>(top[t2], c, 0);
                                    c = lmax;
                                }
                                if (kq > 64) hi = sorted_insert<64>(hi, c, 0);
                            } else {
                                top[t2 / QPR] = sorted_insert<KC>(top[t2 / QPR], c, KC * (t2 % QPR));
                            }
                        }
                        uint32_t nthr = 0u;
                        if constexpr (KC == 128) {
                            if (kq > 64) hdst[lane] = hi;
                            nthr = (uint32_t)((kq <= 64 ? readlane_u64(top[t2], kq - 1) : readlane_u64(hi, kq - 65)) >> 32);
                        } else {
                            nthr = kq > 0 ? (uint32_t)(readlane_u64(top[t2 / QPR], KC * (t2 % QPR) + kq - 1) >> 32) : 0u;
                        }
                        // publish a full list's k-th key value for the query's other work items (the
                        // query index is read while the whole wave is active)
                        const int qt = __builtin_amdgcn_readlane(qg, t2);
                        if (lane == 0 && nthr != 0xFFFFFFFFu)
                            __hip_atomic_fetch_min(gthr + qt, nthr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        if (qcol == t2) {
                            thr = nthr;
                            thr_f = METRIC == 0 ? from_ord(thr) : from_ord(~thr);
                        }
                    }
                }
            }
            // move the unprocessed tail (< 64 pairs) to the front
            const int rest = qn - nproc;
            const uint32_t v = lane < rest ? pq[nproc + lane] : 0u;
            __syncthreads();
            if (lane < rest) pq[lane] = v;
            qn = rest;
        }
        __syncthreads();   // queue writes of this step before the next step's appends
    }
    SIVF_ITEM_SLOT(MQ)
    if constexpr (KC == 128) {
#pragma unroll
        for (int t = 0; t < MQ; t++) {
            if (t < nt) {
                uint64_t *dst = partials + (slot0 + (int64_t)t * nc) * kcap;
                dst[lane] = top[t];
                if (!((hset >> t) & 1u)) dst[64 + lane] = ~0ull;   // no rank 64..127 key yet
            }
        }
    } else {
#pragma unroll
        for (int t = 0; t < MQ; t++)
            if (t < nt && (lane >> (KC == 64 ? 6 : 4)) == (KC == 64 ? 0 : t % QPR) && (lane & (KC - 1)) < kcap)
                partials[(slot0 + (int64_t)t * nc) * kcap + (lane & (KC - 1))] = top[t / QPR];
    }
    SIVF_ITEM_LOOP_END
}

void launch_search_scan_mfma(hipStream_t st, const Dev &S, const SearchBufs &W, int nq, const float *q,
                             int np_stride, int kcap, int k, int kmul, const int32_t *k_per_query) {
    const int npairs = nq * np_stride;
    // k-blocks of 32 dimensions held as B operands: 2, 3, 4 or 8 (d <= 256)
    const int nkb = (S.d + 31) / 32;
#define SIVF_LAUNCH_MFMA_P(M, D, K, P)                                                                       \
    hipLaunchKernelGGL((k_scan_mfma<M, D, K, P>), dim3(scan_grid(k_scan_mfma<M, D, K, P>, S, W, npairs, 0)),    \
                       dim3(64), 0, st, S, W.item_list, W.item_tile, W.item_chunk, W.list_pairs, q, np_stride,  \
                       kcap, k, kmul, k_per_query, W.partials, W.gthr)
#define SIVF_LAUNCH_MFMA(M, D, K)                                                                            \
    do {                                                                                                     \
        if (S.persistent) SIVF_LAUNCH_MFMA_P(M, D, K, true);                                                 \
        else SIVF_LAUNCH_MFMA_P(M, D, K, false);                                                             \
    } while (0)
#define SIVF_LAUNCH_MFMA_K(M, D)                                                                             \
    do {                                                                                                     \
        if (nkb <= 2) SIVF_LAUNCH_MFMA(M, D, 2);                                                             \
        else if (nkb == 3) SIVF_LAUNCH_MFMA(M, D, 3);                                                        \
        else if (nkb == 4) SIVF_LAUNCH_MFMA(M, D, 4);                                                        \
        else SIVF_LAUNCH_MFMA(M, D, 8);                                                                      \
    } while (0)
    if (S.metric == 0 && S.storage == 1) SIVF_LAUNCH_MFMA_K(0, 1);
    else if (S.metric == 0) SIVF_LAUNCH_MFMA_K(0, 2);
    else if (S.storage == 1) SIVF_LAUNCH_MFMA_K(1, 1);
    else SIVF_LAUNCH_MFMA_K(1, 2);
#undef SIVF_LAUNCH_MFMA_K
#undef SIVF_LAUNCH_MFMA
#undef SIVF_LAUNCH_MFMA_P
}

template <int METRIC, int NB, int KC>
static void launch_cert_nb(hipStream_t st, const Dev &S, const SearchBufs &W, const float *q, int np_stride,
                           int kcap, int k, const int32_t *kpq, int npairs) {
    const size_t smem = (size_t)MQ * (S.dp4 + 1) * sizeof(float4);
#define SIVF_LAUNCH_CERT(P)                                                                                  \
    hipLaunchKernelGGL((k_scan_cert<METRIC, NB, P, KC>), dim3(scan_grid(k_scan_cert<METRIC, NB, P, KC>, S, W, npairs, smem)), \
                       dim3(64), smem, st, S, W.item_list, W.item_tile, W.item_chunk, W.list_pairs, q, np_stride, \
                       kcap, k, kpq, W.partials, W.gthr)
    if (S.persistent) SIVF_LAUNCH_CERT(true);
    else SIVF_LAUNCH_CERT(false);
#undef SIVF_LAUNCH_CERT
}

template <int METRIC>
static void launch_cert(hipStream_t st, const Dev &S, const SearchBufs &W, const float *q, int np_stride, int kcap,
                        int k, const int32_t *kpq, int npairs) {
    // blocks of 16 dimensions held as B operands (d <= 256)
    // sorted lists of 16 keys (kcap 16: four queries per register), 64 (kcap 32, 64) or
    // 128 (kcap 128: ranks 64..127 in the partial slot)
    const int nb = (S.d + 15) / 16;
#define SIVF_CERT_NB(KC)                                                                                     \
    do {                                                                                                     \
        if (nb <= 2) launch_cert_nb<METRIC, 2, KC>(st, S, W, q, np_stride, kcap, k, kpq, npairs);            \
        else if (nb <= 4) launch_cert_nb<METRIC, 4, KC>(st, S, W, q, np_stride, kcap, k, kpq, npairs);       \
        else if (nb <= 8) launch_cert_nb<METRIC, 8, KC>(st, S, W, q, np_stride, kcap, k, kpq, npairs);       \
        else launch_cert_nb<METRIC, 16, KC>(st, S, W, q, np_stride, kcap, k, kpq, npairs);                   \
    } while (0)
    if (kcap <= 16) SIVF_CERT_NB(16);
    else if (kcap <= 64) SIVF_CERT_NB(64);
    else SIVF_CERT_NB(128);
#undef SIVF_CERT_NB
}

void launch_scan_cert(hipStream_t st, const Dev &S, const SearchBufs &W, const float *q, int np_stride, int kcap,
                      int k, const int32_t *k_per_query, int npairs) {
    if (S.metric == 0) launch_cert<0>(st, S, W, q, np_stride, kcap, k, k_per_query, npairs);
    else launch_cert<1>(st, S, W, q, np_stride, kcap, k, k_per_query, npairs);
}

}  // namespace sivf
