// The reduced-precision scan (bf16 / fp16 slabs).  Work items, partial lists and
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

}  // namespace sivf
