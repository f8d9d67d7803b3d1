// The certified FP32 scan (one source per metric instantiates it: the variants
// compile in parallel).
#pragma once

#include "scan_dev.h"

namespace sivf {

// Insert key c into a list sorted ascending across the first KC lanes (lane i
// holds the i-th smallest); the largest key drops out and the other lanes keep
// theirs.  Keys are distinct.
template <int KC>
__device__ __forceinline__ uint64_t sorted_insert(uint64_t a, uint64_t c) {
    const int lane = lane_id();
    // previous lane's key: DPP wave_shr:1 (lane 0 keeps its own, unused)
    const uint32_t plo = (uint32_t)__builtin_amdgcn_update_dpp((int)(uint32_t)a, (int)(uint32_t)a, 0x138, 0xf, 0xf, false);
    const uint32_t phi = (uint32_t)__builtin_amdgcn_update_dpp((int)(uint32_t)(a >> 32), (int)(uint32_t)(a >> 32), 0x138,
                                                                0xf, 0xf, false);
    const uint64_t prev = ((uint64_t)phi << 32) | plo;
    const uint64_t r = a < c ? a : ((lane == 0 || prev < c) ? c : prev);
    return (KC == 64 || lane < KC) ? r : a;
}

// Canonical FP32 value of one (row, query) pair, exactly as the VALU scan
// computes it (one fma per dimension, ascending, over the padded chunks);
// eight chunks of loads in flight.  qv4: the query's zero-padded row in LDS.
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
    for (; c0 + 8 <= dp4; c0 += 8) {
        float4 xv[8];
#pragma unroll
        for (int u = 0; u < 8; u++) xv[u] = xp[(int64_t)(c0 + u) * C];
#pragma unroll
        for (int u = 0; u < 8; u++) cert_chunk<METRIC>(r, qv4[c0 + u], xv[u]);
    }
    for (; c0 < dp4; c0++) cert_chunk<METRIC>(r, qv4[c0], xp[(int64_t)c0 * C]);
    return r;
}

// The k-th smallest upper bound v + e among a step's candidates of a query without a
// k-th value (lanes qcol + 16 i hold them), by bisection: at least k candidates lie
// at or below it, so the k best do too.  Returns it for the warm lanes' queries with k
// candidates or more, thd otherwise.  Every lane must call it.
__device__ __forceinline__ float cert_warm(const float (&vv)[16], const float (&ee)[16], uint32_t vm, int kq, bool warm,
                                           float thd) {
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
    return warm && nv >= kq ? hi : thd;
}

// What a work item keeps in LDS beside its query rows: the
// sorted exact keys of each query (ranks 0 .. KL - 1), its k, index and published
// or own k-th key, and the queue of pairs to recompute (window position << 4 |
// query).  Lists in registers need every query's insertion unrolled, and took
// the registers that hold the rows in flight.
constexpr int FQ = 64 + 256;   // queue: fewer than 64 carried over, one row group of 16 x 16 pairs
template <int KL>
struct CertLds {
    uint64_t list[MQ * KL];
    uint32_t pq[FQ];
    uint32_t thr[MQ];
    int kq[MQ], qi[MQ];
};

// Recompute the first nproc queued pairs, one per lane and 64 per round, insert
// the exact keys into their queries' sorted lists, publish and note the new
// thresholds, and move the rest (fewer than 64) to the front.
// KC = 128: ranks 64..127 of a query with k > 64 live in the upper half of its
// partial slot (slot0 + t nc); hset: the queries whose upper half has been written.
template <int METRIC, int KC, int KL>
__device__ __forceinline__ void cert_process(const Dev &S, int nproc, int &qn, CertLds<KL> &F, const float4 *sqr,
                                             int qs, int wslab, int cs, int cm, uint32_t &hset, uint64_t *partials,
                                             uint32_t *gthr, int kcap, int64_t slot0, int nc) {
    const int lane = lane_id(), C = cm + 1, dp4 = S.dp4;
    __syncthreads();
    for (int r0 = 0; r0 < nproc; r0 += 64) {
        const bool act = r0 + lane < nproc;
        const uint32_t e = F.pq[act ? r0 + lane : r0];
        const int t = (int)(e & 15), pw = (int)(e >> 4);
        const int slab = __shfl(wslab, pw >> cs), slot = pw & cm;
        uint64_t key = ~0ull;
        if (act) {
            const float r = cert_exact<METRIC>(S.data + (int64_t)slab * dp4 * C + slot, C, dp4, sqr + t * qs);
            key = ((uint64_t)key_hi<METRIC>(r) << 32) | S.sids[(int64_t)slab * C + slot];
        }
        uint64_t rem = ballot(act);
        while (rem) {   // one query after another
            const int t2 = readlane_i(t, (int)__builtin_ctzll(rem));
            uint64_t bm = ballot(act && t == t2);
            rem &= ~bm;
            const int kq = __builtin_amdgcn_readfirstlane(F.kq[t2]);   // > 0: only live queries have pairs
            uint64_t a = lane < KL ? F.list[t2 * KL + lane] : ~0ull, hi = ~0ull;
            uint64_t *hdst = nullptr;
            if (KC == 128 && kq > 64) {
                hdst = partials + (slot0 + (int64_t)t2 * nc) * kcap + 64;
                if ((hset >> t2) & 1u) hi = hdst[lane];
            }
            // only keys below the query's current k-th key can change its k best
            const uint64_t kth = (KC == 128 && kq > 64) ? readlane_u64(hi, kq - 65) : readlane_u64(a, kq - 1);
            bm &= ballot(key < kth);
            if (!bm) continue;
            while (bm) {
                const int src = (int)__builtin_ctzll(bm);
                bm &= bm - 1;
                uint64_t c = readlane_u64(key, src);
                if (KC == 128) {
                    // a key below the low half's largest enters it and pushes that one down
                    const uint64_t lmax = readlane_u64(a, 63);
                    if (c < lmax) {
                        a = sorted_insert<64>(a, c);
                        c = lmax;
                    }
                    if (kq > 64) hi = sorted_insert<64>(hi, c);
                } else {
                    a = sorted_insert<KC>(a, c);
                }
            }
            if (lane < KL) F.list[t2 * KL + lane] = a;
            if (KC == 128 && kq > 64) {
                hdst[lane] = hi;
                hset |= 1u << t2;
            }
            const uint32_t nthr =
                (uint32_t)(((KC == 128 && kq > 64) ? readlane_u64(hi, kq - 65) : readlane_u64(a, kq - 1)) >> 32);
            if (lane == 0 && nthr != 0xFFFFFFFFu) {   // a full list: publish for the query's other work items
                F.thr[t2] = nthr;
                __hip_atomic_fetch_min(gthr + F.qi[t2], nthr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
    }
    const int rest = qn - nproc;
    const uint32_t v = lane < rest ? F.pq[nproc + lane] : 0u;
    __syncthreads();
    if (lane < rest) F.pq[lane] = v;
    qn = rest;
    __syncthreads();
}

// ------------------------------------------------ certified FP32 scan
//
// FP32 slabs with results identical to the canonical scan.  The matrix cores give
// approximate values for 16 slots x 16 queries: Dt = |x|^2 + |q|^2 - 2 x.q (L2) or
// -x.q (IP, as a distance).  A slot can be among a query's k best only if Dt - e is
// at most the query's current k-th best canonical value; only those pairs get their
// canonical FP32 distance recomputed (sequential fma over ascending dimensions,
// exactly as the VALU scan computes it) and inserted into the query's sorted
// list.  Two filters, each with its half-width e:
//
// Every step: v_mfma_f32_16x16x32_bf16 does 16 times the work per cycle of
// the FP32 form, and few pairs of a query with most of its lists come near its
// top-k.  The slab rows are rounded to bf16 as they arrive (one v_cvt_pk_bf16_f32
// per two values), the queries are held as bf16 pairs hi + lo.  x = xh + xr with
// |xr| <= 2^-8 |x| per component (8 significant bits, round to nearest even) and q =
// qh + ql + qr with |qr| <= 2^-16 |q|, so x.q differs from xh.(qh + ql) by at most
// (2^-8 + 2^-15) |x||q|; the products are exact in fp32, and the 2d + 1 sums (the accumulator
// starts at the row's share of the threshold) add at most two units 2^-24 each of
// |x||q| + |x|^2 / 2.  With N = |x|^2 + |q|^2 >= 2 |x||q|: L2 counts the dot product
// twice, 1.02 2^-8 N + (8d + 16) 2^-24 N, and (3d + 6) 2^-24 N cover the norms and the
// canonical sum; IP half of the former.  Values flushed below 2^-126 are inside the
// additive terms.  Dt - e <= threshold is rearranged as acc >= b_q with acc = dot -
// a_x: a_x (row) is the accumulator's start, b_q (query) moves with the threshold, and
// a lane takes one maximum over its 16 slots.
//
// With the rows' low part too (a step with no threshold yet, or with more than
// FILT_MAX pairs past the first filter, from the rows again): what is left out of xh.(qh
// + ql) + xl.qh is at most 3 2^-16 |x||q|, and the 3d + 1 sums add two units each,
// 1.1 3 2^-16 N + (16d + 96) 2^-24 N for L2, half for IP.  Norms past 2^124 (a sum could
// overflow) send every pair of the step to the recomputation.
// Before a query has k exact values (the first step of a work item), its threshold
// is the k-th smallest upper bound Dt + e among the step's candidates.
//
// Layout.  A operand (lane l): slot l % 16 of the row group, 8 dimensions from
// 32 b + 8 (l / 16), two float4 loads; B the same dimensions of query l % 16.  C (lane l): slots 4 (l / 16) .. +3, query l %
// 16.  Passing pairs are queued in LDS and recomputed one per lane, in full rounds of
// 64 (the queue drains early when a query has no k-th value yet, before the slab
// window moves, and at the end of the item).  Sorted lists of KC keys per query:
// 16 or 64 in LDS; KC = 128 (k up to 128): ranks 0..63 there, ranks 64..127 only for
// queries whose k exceeds 64, in the upper half of the query's own partial slot (read
// and written back by the inserting lanes, each its own rank); a key that enters the
// low half pushes its largest key down into the high half.
//
// What bounds it: the reads, all from the L2 (a list is read once per 16 queries).
// 10,000 queries x 32 of 1,024 lists (1M x 128, 785M pairs): 1.67 ms, the loop
// without passing pairs 1.12 ms = 22 TB/s; on the FP32 MFMA form alone 2.79 ms (half
// of its 1.3 ms matrix-core floor was waiting).  Tiles of 32 queries would halve the
// reads but need 64 registers for the queries and spilled (3.0 ms; with the queries
// in one bf16 term 2.4 ms).
constexpr int FILT_MAX = 48;
typedef float f32x8_t __attribute__((ext_vector_type(8)));
__device__ __forceinline__ f32x8_t join8(float4 a, float4 b) {
    return f32x8_t{a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
}

template <int METRIC, int NKB, bool PERS, int KC, int MODE>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2, 8))) void k_scan_cert(
    Dev S, const int32_t *__restrict__ item_list, const int32_t *__restrict__ item_tile,
    const int32_t *__restrict__ item_chunk, const int32_t *__restrict__ list_pairs, const float *__restrict__ q,
    int np_stride, int kcap, int k, const int32_t *__restrict__ kpq, uint64_t *__restrict__ partials,
    uint32_t *__restrict__ gthr) {
    constexpr int KL = KC == 16 ? 16 : 64;
    constexpr int PF = NKB == 3 ? 3 : (NKB == 1 ? 1 : 2);   // k-blocks of rows in flight (divides NKB)
    extern __shared__ float4 sqr[];   // the tile's 16 query rows, zero-padded to dp4 chunks, stride dp4 + 1
    __shared__ CertLds<KL> F;
    const int lane = threadIdx.x, qcol = lane & 15, kgrp = lane >> 4;
    const int d = S.d, C = S.C, dp4 = S.dp4, sh = S.ctl[CTL_CHUNK];
    const int qs = dp4 + 1;   // LDS row stride: rows start in different banks
    const int cs = __builtin_ctz(C), cm = C - 1;   // slab capacities are powers of two
    // half-widths: first filter h1 N + h0, second l1 N + h0
    const float ca = sqrtf((float)d) * 0x1p-122f, cb = (float)d * 0x1p-120f;
    const float h1 = (METRIC == 0 ? 1.02f * 0x1p-8f + (12.0f * d + 64.0f) * 0x1p-24f
                                  : 1.02f * 0x1p-9f + (6.0f * d + 32.0f) * 0x1p-24f) + 2.f * ca;
    const float l1 = (METRIC == 0 ? 3.3f * 0x1p-16f + (16.0f * d + 96.0f) * 0x1p-24f
                                  : 1.7f * 0x1p-16f + (8.0f * d + 48.0f) * 0x1p-24f) + 2.f * ca;
    const float h0 = 2.f * (ca + cb);
    // accumulator start per unit of |x|^2: minus the row's share of the threshold
    const float ax = METRIC == 0 ? -0.5f * (1.f - h1) : h1;
    SIVF_ITEM_LOOP_BEGIN
    SIVF_ITEM_DECODE(MQ)
    __syncthreads();
    if (lane < MQ) {
        const int qi = pairs[lane < nt ? lane : 0] / np_stride;
        const int kq = lane < nt ? min(query_k(kpq, k, qi), kcap) : 0;
        F.kq[lane] = kq;
        F.qi[lane] = qi;
        F.thr[lane] = kq > 0 ? 0xFFFFFFFFu : 0u;
    }
    for (int i = lane; i < MQ * KL; i += 64) F.list[i] = ~0ull;
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
    // query qcol: |q|^2 and the bf16 operands (dims 32 kb + 8 kgrp .. +8)
    const int qg = F.qi[qcol];
    float qn2 = 0.f;
    uint4 bh[NKB], bl[NKB];
#pragma unroll
    for (int kb = 0; kb < NKB; kb++) {
        const int ch = 8 * kb + 2 * kgrp;
        const float4 z = make_float4(0.f, 0.f, 0.f, 0.f);
        const f32x8_t v = join8(ch < dp4 ? sqr[qcol * qs + ch] : z, ch + 1 < dp4 ? sqr[qcol * qs + ch + 1] : z);
#pragma unroll
        for (int e = 0; e < 8; e++) qn2 = fmaf(v[e], v[e], qn2);
        const bf16x8_t hi = __builtin_convertvector(v, bf16x8_t);
        const f32x8_t rest = v - __builtin_convertvector(hi, f32x8_t);
        bh[kb] = __builtin_bit_cast(uint4, hi);
        bl[kb] = __builtin_bit_cast(uint4, __builtin_convertvector(rest, bf16x8_t));
    }
    qn2 += __shfl_xor(qn2, 16);
    qn2 += __shfl_xor(qn2, 32);
    __syncthreads();
    const bool live = qcol < nt && F.kq[qcol] > 0;
    uint32_t thr = F.thr[qcol];   // high word of query qcol's k-th exact key
    // the k-th exact value in distance space (NaN: none yet, all pass) -> the bf16 filter's bound
    auto dist_of = [&](uint32_t th) { return METRIC == 0 ? from_ord(th) : -from_ord(~th); };
    float bq;
    auto set_bound = [&]() {
        const float thd = dist_of(thr);
        bq = METRIC == 0 ? 0.5f * ((1.f - h1) * qn2 - h0 - thd) : -thd - h0 - h1 * qn2;
    };
    set_bound();
    auto refresh = [&]() {   // this wave's own lists may have tightened it
        const uint32_t own = F.thr[qcol];
        thr = own < thr ? own : thr;
        set_bound();
    };
    const bool item_big = ballot(live && !(qn2 < 0x1p124f)) != 0;
    SIVF_ITEM_SLOT(MQ)
    uint32_t hset = 0;   // KC = 128: queries whose ranks 64..127 have been written to their slot
    auto process = [&](int nproc, int &qn, int wslab) {
        cert_process<METRIC, KC>(S, nproc, qn, F, sqr, qs, wslab, cs, cm, hset, partials, gthr, kcap, slot0, nc);
    };

    const int nslab = (len + cm) >> cs;
    int wbase = -(1 << 30), wslab = 0;   // lane j holds the slab of ordinal wbase + j
    int qn = 0;                          // queued pairs (fewer than 64 carry over to the next step)
    // A operands of row group rg: slot 16 rg + qcol, chunks 8 kb + 2 kgrp, +1 (past the row: its last chunk
    // again, their B lanes are zero); norms of the positions 16 rg + 4 kgrp .. +3 of this lane's results.
    // Work items start at multiples of 64.  MODE 0 (C >= 64): the 64 positions lie in one slab, so
    // every load has a scalar base, one of two 32-bit lane offsets and a constant; MODE 1 (C of 16 or 32):
    // the same per row group.  Positions past the item read other slots of the pool there (any bits
    // in them stay in their own result rows, which are masked).  MODE 2 (C of 4 or 8): each lane has its
    // row's address, and positions past the item read its last rows.
    constexpr int NW = MODE == 0 ? 1 : 4;
    struct Where {
        const char *row[NW], *xn[NW];
    };
    auto locate = [&](int base, Where &w) {
#pragma unroll
        for (int rg = 0; rg < NW; rg++) {
            int64_t row, pos;
            if (MODE < 2) {
                const int b = base + 16 * rg;
                const int64_t slab = __builtin_amdgcn_readlane(wslab, (b >> cs) - wbase);
                row = slab * dp4 * C + (b & cm);
                pos = slab * C + (b & cm);
            } else {
                const int p = base + 16 * rg + qcol, pc = p < p1 ? p : p1 - 1;
                row = (int64_t)__shfl(wslab, (pc >> cs) - wbase) * dp4 * C + (pc & cm);
                const int r = base + 16 * rg + 4 * kgrp, rc = r < p1 ? r : ((p1 - 1) & ~3);
                pos = (int64_t)__shfl(wslab, (rc >> cs) - wbase) * C + (rc & cm);
            }
            w.row[rg] = reinterpret_cast<const char *>(S.data + row);
            w.xn[rg] = reinterpret_cast<const char *>(S.xnorm + pos);
        }
    };
    // byte offsets of the lane's two chunks in a k-block, and in the last one (clamped to the row)
    const uint32_t slot = MODE < 2 ? 16u * qcol : 0u;
    const uint32_t o0 = 32u * kgrp * C + slot, o1 = o0 + 16u * C;
    const uint32_t z0 = 16u * min(8 * (NKB - 1) + 2 * kgrp, dp4 - 1) * C + slot;
    const uint32_t z1 = 16u * min(8 * (NKB - 1) + 2 * kgrp + 1, dp4 - 1) * C + slot;
    const uint32_t on = MODE < 2 ? 16u * kgrp : 0u;
    auto row_at = [&](const Where &w, int rg) { return MODE == 0 ? w.row[0] + 256 * rg : w.row[rg % NW]; };
    auto fetch = [&](int kb, const Where &w, float4 (&a)[4][2]) {
        const bool z = kb == NKB - 1;
#pragma unroll
        for (int rg = 0; rg < 4; rg++) {
            const char *b = row_at(w, rg) + (z ? 0 : 128 * kb * C);
            a[rg][0] = *reinterpret_cast<const float4 *>(b + (z ? z0 : o0));
            a[rg][1] = *reinterpret_cast<const float4 *>(b + (z ? z1 : o1));
        }
    };
    auto norms = [&](const Where &w, float4 (&xn)[4]) {
#pragma unroll
        for (int rg = 0; rg < 4; rg++)
            xn[rg] = *reinterpret_cast<const float4 *>((MODE == 0 ? w.xn[0] + 64 * rg : w.xn[rg % NW]) + on);
    };
    float4 ab[PF][4][2], xn4[4];
    Where at0, at1;       // this step's and the next one's rows
    bool ahead = false;   // this step's first PF k-blocks and norms are already in flight
    uint32_t pub = ~0u;
    for (int base = p0; base < p1; base += 64) {
        const int last_ord = min(base + 63, p1 - 1) >> cs;
        if (last_ord >= wbase + 64) {
            wbase = base >> cs;
            wslab = (wbase + lane < nslab) ? slab_of(S, l, wbase + lane) : 0;
            __builtin_amdgcn_s_waitcnt(0);   // here, so that no later step waits for its prefetched rows instead
        }
        // every fourth step: the best k-th key any work item has published for this query (those k keys are
        // real candidates, so nothing behind it can enter the query's final k; a stale one only filters less)
        const bool look = ((base - p0) & 255) == 0;
        if (look) pub = live ? __hip_atomic_load(gthr + qg, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : ~0u;
        if (!ahead) {
            locate(base, at0);
            norms(at0, xn4);
#pragma unroll
            for (int i = 0; i < PF; i++) fetch(i, at0, ab[i]);
        }
        const int nb = base + 64;
        const bool moves = (min(nb + 63, p1 - 1) >> cs) >= wbase + 64;   // the next step moves the slab window
        const bool next = nb < p1 && !moves;
        if (nb > p1) {   // norms past the item are those of other slots
#pragma unroll
            for (int rg = 0; rg < 4; rg++) {
                const int left = p1 - (base + 16 * rg + 4 * kgrp);
                xn4[rg].x = left > 0 ? xn4[rg].x : 0.f;
                xn4[rg].y = left > 1 ? xn4[rg].y : 0.f;
                xn4[rg].z = left > 2 ? xn4[rg].z : 0.f;
                xn4[rg].w = left > 3 ? xn4[rg].w : 0.f;
            }
        }
        f32x4_t acc[4];
        uint32_t xmax = 0;   // norms are not negative: their bits order as they do
#pragma unroll
        for (int rg = 0; rg < 4; rg++) {
            acc[rg] = f32x4_t{ax * xn4[rg].x, ax * xn4[rg].y, ax * xn4[rg].z, ax * xn4[rg].w};
            xmax = max(max(xmax, max(__float_as_uint(xn4[rg].x), __float_as_uint(xn4[rg].y))),
                       max(__float_as_uint(xn4[rg].z), __float_as_uint(xn4[rg].w)));
        }
        locate(next ? nb : base, at1);   // without a next step in reach: this one's rows again, unused
#pragma unroll
        for (int kb = 0; kb < NKB; kb++) {
            float4(&a)[4][2] = ab[kb % PF];
            uint4 ah[4];
#pragma unroll
            for (int rg = 0; rg < 4; rg++)
                ah[rg] = __builtin_bit_cast(uint4, __builtin_convertvector(join8(a[rg][0], a[rg][1]), bf16x8_t));
            if (kb + PF < NKB) fetch(kb + PF, at0, a);
            else fetch(kb + PF - NKB, at1, a);
#pragma unroll
            for (int rg = 0; rg < 4; rg++) acc[rg] = mfma_16x16x32<1>(ah[rg], bh[kb], acc[rg]);
#pragma unroll
            for (int rg = 0; rg < 4; rg++) acc[rg] = mfma_16x16x32<1>(ah[rg], bl[kb], acc[rg]);
        }
        norms(at1, xn4);
        if (look && pub < thr) {
            thr = pub;
            set_bound();
        }
        const bool big = item_big || ballot(xmax >= __float_as_uint(0x1p124f)) != 0;
        float m = acc[0][0];
#pragma unroll
        for (int i = 1; i < 16; i++) m = fmaxf(m, acc[i >> 2][i & 3]);
        ahead = next;
        if (ballot(big || (live && !(m < bq)))) {
            // bit 4 rg + j: position 16 rg + 4 kgrp + j in range and (lazy deletes) live
            const uint32_t vm = lane_valid16(step_valid(S, base, p1, wslab, wbase, cs, cm), kgrp);
            uint32_t pmask = 0;
#pragma unroll
            for (int i = 0; i < 16; i++) pmask |= (!(acc[i >> 2][i & 3] < bq) ? 1u : 0u) << i;
            if (big) pmask = 0xFFFFu;
            if (!live) pmask = 0;
            pmask &= vm;
            int incl = wave_incl_scan_dpp(__builtin_popcount(pmask));
            int total = __builtin_amdgcn_readlane(incl, 63);
            const bool warm = live && thr == 0xFFFFFFFFu;
            if (!big && (total > FILT_MAX || (total > 0 && ballot(warm)))) {
                // the rows' low parts, from the rows again (they are in the caches)
                float vv[16], ee[16];
                float4 xr4[4];
                norms(at0, xr4);
#pragma unroll
                for (int kb = 0; kb < NKB; kb++) {
                    float4 t[4][2];
                    fetch(kb, at0, t);
#pragma unroll
                    for (int rg = 0; rg < 4; rg++) {
                        const f32x8_t v = join8(t[rg][0], t[rg][1]);
                        const bf16x8_t hi = __builtin_convertvector(v, bf16x8_t);
                        const f32x8_t rest = v - __builtin_convertvector(hi, f32x8_t);
                        acc[rg] = mfma_16x16x32<1>(__builtin_bit_cast(uint4, __builtin_convertvector(rest, bf16x8_t)),
                                                   bh[kb], acc[rg]);
                    }
                }
#pragma unroll
                for (int rg = 0; rg < 4; rg++) {
                    const float xs[4] = {xr4[rg].x, xr4[rg].y, xr4[rg].z, xr4[rg].w};
#pragma unroll
                    for (int j = 0; j < 4; j++) {
                        const float sq = qn2 + xs[j], dot = acc[rg][j] - ax * xs[j];
                        vv[4 * rg + j] = METRIC == 0 ? fmaf(-2.f, dot, sq) : -dot;
                        ee[4 * rg + j] = fmaf(l1, sq, h0);
                    }
                }
                float thd = dist_of(thr);
                if (ballot(warm)) thd = cert_warm(vv, ee, vm, F.kq[qcol], warm, thd);
                uint32_t pm = 0;
#pragma unroll
                for (int i = 0; i < 16; i++) pm |= (!(vv[i] - ee[i] > thd) ? 1u : 0u) << i;
                pmask &= pm;
                incl = wave_incl_scan_dpp(__builtin_popcount(pmask));
                total = __builtin_amdgcn_readlane(incl, 63);
            }
            // queue the pairs (a row group at a time where they would not fit) and recompute full rounds
            // of 64; everything when a query still waits for its first k-th value
            const int parts = total > FQ - 64 ? 4 : 1;
            for (int pt = 0; pt < parts && total > 0; pt++) {
                uint32_t mine = pmask;
                if (parts > 1) {
                    mine &= 0xFu << (4 * pt);
                    incl = wave_incl_scan_dpp(__builtin_popcount(mine));
                }
                int at = qn + incl - __builtin_popcount(mine);
                qn += __builtin_amdgcn_readlane(incl, 63);
                const int wpos = base - (wbase << cs);   // queued positions are relative to the slab window
                while (mine) {
                    const int bit = __builtin_ctz(mine);
                    mine &= mine - 1;
                    F.pq[at++] = ((uint32_t)(wpos + 16 * (bit >> 2) + 4 * kgrp + (bit & 3)) << 4) | (uint32_t)qcol;
                }
                const int nproc = ballot(warm) ? qn : (qn & ~63);
                if (nproc > 0) process(nproc, qn, wslab);
            }
            refresh();
        }
        if (qn > 0 && (nb >= p1 || moves)) {   // before the slab window moves, and at the end
            process(qn, qn, wslab);
            refresh();
        }
        at0 = at1;
    }
    __syncthreads();
    for (int t = 0; t < nt; t++) {
        uint64_t *dst = partials + (slot0 + (int64_t)t * nc) * kcap;
        if (lane < KL && lane < kcap) dst[lane] = F.list[t * KL + lane];
        if (KC == 128 && !((hset >> t) & 1u)) dst[64 + lane] = ~0ull;   // no rank 64..127 key yet
    }
    SIVF_ITEM_LOOP_END
}

template <int METRIC, int NKB, int KC, int MODE>
static void launch_cert_p(hipStream_t st, const Dev &S, const SearchBufs &W, const float *q, int np_stride, int kcap,
                          int k, const int32_t *kpq, int npairs) {
    const size_t smem = (size_t)MQ * (S.dp4 + 1) * sizeof(float4);
#define SIVF_LAUNCH_CERT(P)                                                                                  \
    hipLaunchKernelGGL((k_scan_cert<METRIC, NKB, P, KC, MODE>),                                               \
                       dim3(scan_grid(k_scan_cert<METRIC, NKB, P, KC, MODE>, S, W, npairs, smem)), dim3(64), smem, st, S, \
                       W.item_list, W.item_tile, W.item_chunk, W.list_pairs, q, np_stride, kcap, k, kpq, W.partials, \
                       W.gthr)
    if (S.persistent) SIVF_LAUNCH_CERT(true);
    else SIVF_LAUNCH_CERT(false);
#undef SIVF_LAUNCH_CERT
}

template <int METRIC>
static void launch_cert(hipStream_t st, const Dev &S, const SearchBufs &W, const float *q, int np_stride, int kcap,
                        int k, const int32_t *kpq, int npairs) {
    // k-blocks of 32 dimensions (d <= 256); sorted lists of 16 keys (kcap 16), 64 (kcap 32, 64) or 128 (kcap 128:
    // ranks 64..127 in the partial slot); row addressing by the slab capacity
    const int nkb = (S.d + 31) / 32;
#define SIVF_CERT_NKB(KC, MODE)                                                                              \
    do {                                                                                                     \
        if (nkb <= 1) launch_cert_p<METRIC, 1, KC, MODE>(st, S, W, q, np_stride, kcap, k, kpq, npairs);      \
        else if (nkb <= 2) launch_cert_p<METRIC, 2, KC, MODE>(st, S, W, q, np_stride, kcap, k, kpq, npairs); \
        else if (nkb <= 3) launch_cert_p<METRIC, 3, KC, MODE>(st, S, W, q, np_stride, kcap, k, kpq, npairs); \
        else if (nkb <= 4) launch_cert_p<METRIC, 4, KC, MODE>(st, S, W, q, np_stride, kcap, k, kpq, npairs); \
        else launch_cert_p<METRIC, 8, KC, MODE>(st, S, W, q, np_stride, kcap, k, kpq, npairs);               \
    } while (0)
#define SIVF_CERT_MODE(KC)                                                                                   \
    do {                                                                                                     \
        if (S.C >= 64) SIVF_CERT_NKB(KC, 0);                                                                 \
        else if (S.C >= 16) SIVF_CERT_NKB(KC, 1);                                                            \
        else SIVF_CERT_NKB(KC, 2);                                                                           \
    } while (0)
    if (kcap <= 16) SIVF_CERT_MODE(16);
    else if (kcap <= 64) SIVF_CERT_MODE(64);
    else SIVF_CERT_MODE(128);
#undef SIVF_CERT_MODE
#undef SIVF_CERT_NKB
}

}  // namespace sivf
