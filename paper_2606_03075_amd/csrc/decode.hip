// Single-query decode attention over the pruned, ragged per-layer cache.
//
// Each decode step appends the new token's key and value to every layer's cache
// (Sec. 3.1, Eq. (3)-(4)) and attends over the b_l retained plus the step + 1
// appended tokens.  This is a pure HBM stream of the cache (one read per step),
// so the kernel is organised for bytes in flight, not for math:
//   * one workgroup per (sequence, layer, KV head[, split]): the KV head's rows
//     are read once and serve all query heads that share it (GQA);
//   * a token row of head_dim bf16 is read by head_dim/8 lanes with 16-byte
//     non-temporal loads; each lane group works on blocks of 4 tokens from two
//     register buffers, issuing the next block's K and V loads before consuming
//     the current one (a trip count that is uniform over the workgroup and even,
//     with every load unconditional, so the compiler's waits stay per block);
//   * online softmax per lane group, merged across groups with wave shuffles and
//     across the 4 waves through LDS; when the (sequence, layer, KV head) count is
//     too small to fill the GPU, or a unit is long, the token range is split, and the unit's
//     last workgroup to finish combines the partial (max, sum, weighted sum) triples
//     (unit_splits, split_unit, combine_splits).
// The step's new token is read from the k_new / v_new inputs (the cache slot it
// is written to is not re-read in the same launch).  The cache is either one
// contiguous segment per (sequence, layer) or fixed-size pages found through a
// block table (staged in LDS); with per-sequence steps (continuous batching) a
// sequence whose step is outside [0, reserve) is skipped.  An optional unit order
// (from the budget call: longest segments first) sets which (sequence, layer) each
// workgroup serves, so the long segments do not all start last.
#include <algorithm>
#include <atomic>
#include <chrono>
#include <climits>
#include <mutex>

#include "tgvkv_device.h"
#include "tgvkv_rows.h"
#include "tgvkv_shape.h"

namespace tgvkv {
namespace {

constexpr int kThreads = 256;
// query heads per KV head from which decode runs on the matrix cores
constexpr int kMfmaMinGroup = 3;
constexpr int kMaxSplits = 8;  // of a unit's token range
constexpr int kCUs = 256;
constexpr int kMaxSplitGroups = 1024;  // workgroups of the units' splits, about

__device__ __forceinline__ void unpack8(u32x4 r, float (&f)[8]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        f[2 * i] = __uint_as_float(r[i] << 16);
        f[2 * i + 1] = __uint_as_float(r[i] & 0xFFFF0000u);
    }
}

// Split partials in one launch: every workgroup of a unit writes its partial, then its mark, then reads
// the unit's marks; one that finds them all combines the partials, in split order, and clears the
// marks.  The workgroup whose mark lands last finds them all, unless another has combined already; two
// that both find them all write the same values.  No workgroup waits for another.  A launch of its own
// for the combination cost 5.4 us of kernel and a gap: one layer of 8 sequences (32 units in 8 splits)
// 14.0 -> 12.3 us per step replayed from a graph, 14.7 -> 11.6 us launched; 32 units of 300 rows, one
// query head each, 14.4 -> 7.7 us.
//
// The marks live in the caller's workspace, whose first contents are unknown, so a mark is the number
// of its call, 64 bits that differ between calls (counted from a scrambled clock).  A replayed graph
// brings the same number again, but the last call on a workspace left its marks cleared.
struct Splits {
    unsigned long long* marks;  // [B*L*H_kv][most], null without a split
    unsigned long long call;    // never 0
    int most, base;             // workgroups per unit; splits of a short unit
    int rows;                   // rows per split of a longer one
    int span;                   // units per 256 workgroups
};

// Splits of a unit of `len` rows (len is known on the device only); called by whole waves, with the same
// arguments in every workgroup of the unit.
//
// The TVB budgets of one call differ by an order of magnitude, and without more splits for its longest units
// these set the time: 160 units of 400 to 4000 rows, mean 1500, one query head: 42.1 us with one workgroup each,
// 30.1 in splits; 132 units of up to 10000 rows, seven query heads, 137 against 59.  A call of even lengths
// gains nothing: 168 units of 1130 rows take 19.5 us whole, 23.2 in three splits each; 400 units of 2000 rows 67
// against 73.  So the units are split only where the longest keeps its CU well beyond the call's mean load of a
// CU (with more units than CUs, the longest and one of mean length): by half and 700 rows, the extra
// partials' cost.  The line lies between 132 units of 2000 rows (28.6 us whole, 33.3 split) and of 4000 rows (52.5
// against 48.4), and 168 units of 810 to 1620 rows (22.9 against 27.9) and of 2870 to 5740 rows (66 against 58.6).
// Reading the lengths costs a call of whole units over kWholeRows 1 to 2 us (the 19.5 us above now 21.0).  A call
// of no unit over kWholeRows is not worth the look (160 units of 700 rows: 13.8 us whole, 16.6 in two).
constexpr int kWholeRows = 1024;
__device__ __forceinline__ int unit_splits(const Splits& sp, const Shape& s, int len, const int32_t* budgets,
                                           const int32_t* steps, int step, int reserve) {
    if (len <= kWholeRows || sp.base == sp.most) return sp.base;
    const int segments = s.B * s.L;
    float longest = 0.f, rows = 0.f;  // of the segments that decode
    for (int i0 = threadIdx.x & 63; i0 < segments; i0 += 256) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int i = min(i0 + 64 * u, segments - 1);
            const int st = steps != nullptr ? steps[i / s.L] : step;
            const float rows_i = (float)(budgets[i] + st + 1);
            if (i0 + 64 * u < segments && st >= 0 && st < reserve) {
                longest = fmaxf(longest, rows_i);
                rows += rows_i;
            }
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        longest = fmaxf(longest, __shfl_xor(longest, o));
        rows += __shfl_xor(rows, o);
    }
    float load = longest / sp.base;
    if (segments * s.Hkv > kCUs) load += rows / segments;
    if (load <= 1.5f * (rows * s.Hkv / kCUs) + 700.f) return sp.base;
    return min(max(sp.base, (len + sp.rows - 1) / sp.rows), sp.most);
}

// The (unit, split) of a workgroup; false for none.  Each 256 workgroups, one per CU, hold every split of
// the next `span` units, split by split.  Long units, which come first in the dispatch order, thus
// spread over every CU; each 256 start `base` splits further on, so that short units' workgroups land
// on CUs of their own, and every other 256 hold their units backwards, which evens the CUs' shares.
// (A unit's splits next to one another left the active ones on a few XCDs when units are short: 112 units
// of 1000 rows 30.4 us against 14.3.)
__device__ __forceinline__ bool split_unit(const Splits& sp, int units, int bid, int& unit, int& split) {
    const int row = bid / kCUs, blk = bid % kCUs / sp.span, j = bid % kCUs % sp.span;
    unit = row * sp.span + ((row & 1) ? sp.span - 1 - j : j);
    split = (blk + sp.most - row * sp.base % sp.most) % sp.most;
    return blk < sp.most && unit < units;
}

// Partials pass between workgroups of different XCDs, whose L2 caches are apart.  They are written and
// read as GPU-scope atomics, which go through to memory, so a finished store (vmcnt) is visible to the
// whole GPU and no cache has to be written back or dropped: with plain stores and a GPU-scope fence
// on either side, whose write-back covers the whole L2, the step took 48 us.  That relies on gfx950, where
// such accesses write and read through; in the language relaxed atomics order nothing between them, so
// the waits in between hold the compiler too (wait_vmem_ordered).
__device__ __forceinline__ void store_shared(float* p, float v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float load_shared(const float* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Called by all threads of a workgroup after they wrote its partial of query heads bh0 .. bh0 + G - 1
// (G <= GMAX).
template <int D, int GMAX>
__device__ __forceinline__ void combine_splits(const Splits& sp, size_t slot, int split, size_t bh0, int G, int nsplit,
                                               const float* ws_part, float* __restrict__ out) {
    constexpr int ITERS = (GMAX * D + kThreads - 1) / kThreads;
    __shared__ int last;
    __shared__ float ml[2][GMAX][kMaxSplits];
    wait_vmem_ordered();  // this thread's part of the partial has reached memory (store_shared) ...
    __syncthreads();  // ... and every thread's has, before the arrival
    const int stride = sp.most;
    unsigned long long* marks = sp.marks + slot * stride;
    if (threadIdx.x < 64) {
        if (threadIdx.x == 0)
            __hip_atomic_store(marks + split, sp.call, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        wait_vmem_ordered();  // the mark has reached memory before the others' are read
        const bool here = threadIdx.x >= nsplit ||
                          __hip_atomic_load(marks + threadIdx.x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == sp.call;
        const bool all = __ballot(!here) == 0;
        if (threadIdx.x == 0) last = all;
    }
    __syncthreads();
    if (!last) return;
    // every load in flight at once: the weighted sums to registers, maxima and sums to LDS
    float a[ITERS][kMaxSplits];
#pragma unroll
    for (int it = 0; it < ITERS; ++it) {
        const int x = min((int)threadIdx.x + it * kThreads, G * D - 1);
        const float* p = ws_part + (bh0 + x / D) * stride * (size_t)(D + 2) + 2 + x % D;
#pragma unroll
        for (int i = 0; i < kMaxSplits; ++i) a[it][i] = load_shared(p + min(i, nsplit - 1) * (D + 2));
    }
    if (threadIdx.x < G * nsplit) {
        const int h = threadIdx.x / nsplit, i = threadIdx.x % nsplit;
        const float* p = ws_part + ((bh0 + h) * stride + i) * (size_t)(D + 2);
        const float m = load_shared(p), l = load_shared(p + 1);
        ml[0][h][i] = m;
        ml[1][h][i] = l;
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < ITERS; ++it) {
        const int x = threadIdx.x + it * kThreads;
        if (x >= G * D) break;
        const int h = x / D;
        float M = kNegInf;
        for (int i = 0; i < nsplit; ++i) M = fmaxf(M, ml[0][h][i]);
        float num = 0.f, den = 0.f;
#pragma unroll
        for (int i = 0; i < kMaxSplits; ++i) {
            if (i < nsplit) {
                const float sc = fast_exp2(ml[0][h][i] - M);
                num += sc * a[it][i];
                den += sc * ml[1][h][i];
            }
        }
        out[(bh0 + h) * D + x % D] = num / den;
    }
    if (threadIdx.x < nsplit)
        __hip_atomic_store(marks + threadIdx.x, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <int D, int GMAX, class Rows, bool SPLIT>
__global__ __launch_bounds__(kThreads) void decode_kernel(Shape s, Rows rows, uint16_t* __restrict__ kc,
                                                          uint16_t* __restrict__ vc,
                                                          const int32_t* __restrict__ budgets, int reserve, int step,
                                                          const int32_t* __restrict__ steps,
                                                          const uint16_t* __restrict__ q,
                                                          const uint16_t* __restrict__ k_new,
                                                          const uint16_t* __restrict__ v_new, float* __restrict__ out,
                                                          float* ws_part, Splits sp,
                                                          const int32_t* __restrict__ unit_order) {
    constexpr int LPR = D / 8;         // lanes per token row
    constexpr int GPW = 64 / LPR;      // lane groups per wave
    constexpr int NGRP = 4 * GPW;      // lane groups per workgroup
    constexpr int kUnroll = 4;  // tokens per lane group in each of the two register buffers
    __shared__ float wm[4][GMAX], wl[4][GMAX];
    __shared__ float wacc[4][GMAX][D];
    extern __shared__ int lds_pages[];  // paged layout: the unit's page ids

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int sub = lane % LPR;
    const int grp = wave * GPW + lane / LPR;
    int bid = blockIdx.x, split = 0;
    if (SPLIT && !split_unit(sp, s.B * s.L * s.Hkv, blockIdx.x, bid, split)) return;
    const int slot = bid;  // the unit's marks
    const int kvh = bid % s.Hkv;
    // dispatch order: unit_order[i] is the (sequence, layer) the i-th group of workgroups serves
    // (clamped, so a wrong order can never address outside the batch)
    const int bl = unit_order != nullptr ? min(max(unit_order[bid / s.Hkv], 0), s.B * s.L - 1) : bid / s.Hkv;
    const int G = s.G;

    // continuous batching: each sequence at its own step, outside [0, reserve) = not decoding
    const int st = steps != nullptr ? steps[bl / s.L] : step;
    if (st < 0 || st >= reserve) return;  // uniform over the workgroup, before any barrier
    const int bsz = budgets[bl];
    const int len = bsz + st + 1;
    const int nsplit = SPLIT ? unit_splits(sp, s, len, budgets, steps, step, reserve) : 1;
    if (SPLIT && split >= nsplit) return;  // uniform, before any barrier
    rows.init(s, bl, kvh, bsz, len, lds_pages);
    __syncthreads();
    const uint16_t* knew = k_new + ((size_t)bl * s.Hkv + kvh) * D;
    const uint16_t* vnew = v_new + ((size_t)bl * s.Hkv + kvh) * D;

    float qv[GMAX][8];  // the scaled query heads, set once the first block's loads are in flight

    const int per = (len + nsplit - 1) / nsplit;
    const int t0 = min(split * per, len), t1 = min(t0 + per, len);

    float m[GMAX], l[GMAX], acc[GMAX][8];
#pragma unroll
    for (int h = 0; h < GMAX; ++h) {
        m[h] = kNegInf;
        l[h] = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[h][e] = 0.f;
    }

    constexpr int S = NGRP * kUnroll;
    // loads of one block of kUnroll tokens per lane group; rows past t1 (and the step's own
    // token) read the fresh k_new / v_new row, so every load is unconditional
    auto issue = [&](u32x4 (&kr)[kUnroll], u32x4 (&vr)[kUnroll], int n0) {
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            const int n = n0 + u * NGRP;
            const bool fresh = n >= len - 1 || n >= t1;
            const size_t r = fresh ? 0 : rows.row(n);
            kr[u] = load16_stream((fresh ? knew : kc + r) + sub * 8);
            vr[u] = load16_stream((fresh ? vnew : vc + r) + sub * 8);
        }
    };
    auto consume = [&](const u32x4 (&kr)[kUnroll], const u32x4 (&vr)[kUnroll], int n0) {
        bool ok[kUnroll];
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) ok[u] = n0 + u * NGRP < t1;
#pragma unroll
        for (int h = 0; h < GMAX; ++h) {
            if (h >= G) continue;
            float z[kUnroll];
            float mx = kNegInf;
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) {
                float kf[8];
                unpack8(kr[u], kf);
                float d = 0.f;
#pragma unroll
                for (int e = 0; e < 8; ++e) d += qv[h][e] * kf[e];
                d = group_sum<LPR>(d);
                z[u] = ok[u] ? d : kNegInf;
                mx = fmaxf(mx, z[u]);
            }
            if (mx > m[h]) {
                const float sc = fast_exp2(m[h] - mx);
                l[h] *= sc;
#pragma unroll
                for (int e = 0; e < 8; ++e) acc[h][e] *= sc;
                m[h] = mx;
            }
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) {
                if (!ok[u]) continue;
                const float p = fast_exp2(z[u] - m[h]);
                float vf[8];
                unpack8(vr[u], vf);
                l[h] += p;
#pragma unroll
                for (int e = 0; e < 8; ++e) acc[h][e] += p * vf[e];
            }
        }
    };
    // two register buffers: the next block's loads are in flight while this block is consumed;
    // the trip count is uniform over the workgroup and even (the extra half only masks)
    const int pairs = (t1 - t0 + 2 * S - 1) / (2 * S);
    u32x4 ka[kUnroll], va[kUnroll], kb[kUnroll], vb[kUnroll];
    int n0 = t0 + grp;
    issue(ka, va, n0);
    {
        // the query's latency overlaps the first block's: wait for it (and only it) here
        u32x4 qr[GMAX];
#pragma unroll
        for (int h = 0; h < GMAX; ++h) {
            const u32x4 z = {0u, 0u, 0u, 0u};
            qr[h] = h < G ? load16(q + ((size_t)bl * s.H + kvh * G + h) * D + sub * 8) : z;
            settle(qr[h]);
        }
#pragma unroll
        for (int h = 0; h < GMAX; ++h) {
            unpack8(qr[h], qv[h]);
#pragma unroll
            for (int e = 0; e < 8; ++e) qv[h][e] *= s.scale2;
        }
    }
    for (int pi = 0; pi < pairs; ++pi) {
        issue(kb, vb, n0 + S);
        consume(ka, va, n0);
        issue(ka, va, n0 + 2 * S);
        consume(kb, vb, n0 + S);
        n0 += 2 * S;
    }
    // the step's token into its cache slot (this launch reads it from k_new / v_new)
    if (split == 0 && tid < LPR) {
        const size_t r = rows.row(bsz + st);
        store16(kc + r + tid * 8, load16(knew + tid * 8));
        store16(vc + r + tid * 8, load16(vnew + tid * 8));
    }

    // merge the lane groups of the wave
#pragma unroll
    for (int h = 0; h < GMAX; ++h) {
        if (h >= G) continue;
#pragma unroll
        for (int off = LPR; off < 64; off <<= 1) {
            const float m2 = shfl_xor(m[h], off), l2 = shfl_xor(l[h], off);
            float a2[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) a2[e] = shfl_xor(acc[h][e], off);
            const float mn = fmaxf(m[h], m2);
            if (mn != kNegInf) {
                const float s1 = fast_exp2(m[h] - mn), s2 = fast_exp2(m2 - mn);
                l[h] = l[h] * s1 + l2 * s2;
#pragma unroll
                for (int e = 0; e < 8; ++e) acc[h][e] = acc[h][e] * s1 + a2[e] * s2;
                m[h] = mn;
            }
        }
        if (lane < LPR) {
            if (lane == 0) {
                wm[wave][h] = m[h];
                wl[wave][h] = l[h];
            }
#pragma unroll
            for (int e = 0; e < 8; ++e) wacc[wave][h][sub * 8 + e] = acc[h][e];
        }
    }
    __syncthreads();
    for (int x = tid; x < G * D; x += kThreads) {
        const int h = x / D, dd = x % D;
        float M = kNegInf;
#pragma unroll
        for (int w = 0; w < 4; ++w) M = fmaxf(M, wm[w][h]);
        float num = 0.f, den = 0.f;
        if (M != kNegInf) {
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                const float sc = fast_exp2(wm[w][h] - M);
                num += sc * wacc[w][h][dd];
                den += sc * wl[w][h];
            }
        }
        const size_t bh = (size_t)bl * s.H + kvh * G + h;
        if (!SPLIT || nsplit == 1) {
            out[bh * D + dd] = num / den;
        } else {
            float* p = ws_part + (bh * sp.most + split) * (size_t)(D + 2);
            store_shared(p + 2 + dd, num);
            if (dd == 0) {
                store_shared(p, M);
                store_shared(p + 1, den);
            }
        }
    }
    if constexpr (SPLIT) {
        if (nsplit > 1)
            combine_splits<D, GMAX>(sp, slot, split, (size_t)bl * s.H + kvh * G, G, nsplit, ws_part, out);
    }
}

// Grouped-query decode on the matrix cores, for several query heads per KV head.
// The VALU kernel above spends each lane group's instructions on one token and
// one head at a time, replicated over the 16 lanes of a row: with G heads its
// work per cached byte grows G-fold and it stops being bound by HBM.  Here a
// 16-token block and all G heads (padded to 16) are one MFMA tile:
//   * the block's K and V rows are loaded whole (16 lanes per 256-byte row) and
//     staged in a per-wave LDS area; read straight into MFMA layout, each quarter
//     wave of a K load would touch 16 rows, 8x the L1 lookups of a row-wise load;
//   * S^T = K Q^T on v_mfma_f32_16x16x32_bf16, keys on the M side: lane l then
//     holds the scores of head l%16 for tokens 4*(l/16) .. +3;
//   * the block max of each head is taken over the lane's 4 values and across
//     the lane quarters, so the 16 lanes of a head share one running max; the
//     output rows are rescaled only when some head's max grew;
//   * O += P V on v_mfma_f32_16x16x16_bf16: the A operand P[head][token] is
//     exactly the lane's 4 probabilities, split into a bf16 high part and a bf16
//     remainder (two MFMAs, about 16 significant bits); the B operand needs
//     V[token][dim] with tokens along k, which the V stage gives: rows padded to
//     272 bytes, so the four lane quarters read rows 4 apart from disjoint banks,
//     and each lane reads one dword (two dims) per token, feeding two 16-dim
//     output blocks;
//   * the 4 waves of a workgroup take alternate 16-token blocks of the split.  One
//     register buffer per wave: as soon as a block's rows are in LDS the next
//     block's loads are issued (unconditional, clamped to the fresh row past the
//     end), so they stream in during the block's softmax and P V.  That keeps the
//     kernel at 122 VGPRs, 4 waves per SIMD; a second buffer cost a wave per SIMD
//     and measured slower.  The waves then merge through LDS as the VALU kernel does.
template <int D, int GMAX, class Rows, bool SPLIT>
__global__ __launch_bounds__(kThreads) void decode_mfma_kernel(Shape s, Rows rows, uint16_t* __restrict__ kc,
                                                               uint16_t* __restrict__ vc,
                                                               const int32_t* __restrict__ budgets, int reserve,
                                                               int step, const int32_t* __restrict__ steps,
                                                               const uint16_t* __restrict__ q,
                                                               const uint16_t* __restrict__ k_new,
                                                               const uint16_t* __restrict__ v_new,
                                                               float* __restrict__ out, float* ws_part, Splits sp,
                                                               const int32_t* __restrict__ unit_order) {
    constexpr int KSTEPS = D / 32;          // k-steps of S^T = K Q^T over the head dim
    constexpr int NB2 = D / 32;             // pairs of 16-dim output blocks
    constexpr int VROWB = D * 2 + 16;       // padded LDS row of the V stage, bytes
    constexpr int VCH = D / 8;              // 16-byte chunks per row
    constexpr int VLOADS = 16 * VCH / 64;   // 16-byte V loads per lane per block
    constexpr int STAGE = 4 * 16 * VROWB * 2;  // per wave: the block's V rows, then its K rows
    constexpr int MERGE = 4 * GMAX * (D + 2) * (int)sizeof(float);
    __shared__ __align__(16) char smem[STAGE > MERGE ? STAGE : MERGE];
    extern __shared__ int lds_pages[];  // paged layout: the unit's page ids

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int c = lane & 15, qq = lane >> 4;
    int bid = blockIdx.x, split = 0;
    if (SPLIT && !split_unit(sp, s.B * s.L * s.Hkv, blockIdx.x, bid, split)) return;
    const int slot = bid;  // the unit's marks
    const int kvh = bid % s.Hkv;
    const int bl = unit_order != nullptr ? min(max(unit_order[bid / s.Hkv], 0), s.B * s.L - 1) : bid / s.Hkv;
    const int G = s.G;

    const int st = steps != nullptr ? steps[bl / s.L] : step;
    if (st < 0 || st >= reserve) return;  // uniform over the workgroup, before any barrier
    const int bsz = budgets[bl];
    const int len = bsz + st + 1;
    const int nsplit = SPLIT ? unit_splits(sp, s, len, budgets, steps, step, reserve) : 1;
    if (SPLIT && split >= nsplit) return;  // uniform, before any barrier
    rows.init(s, bl, kvh, bsz, len, lds_pages);
    __syncthreads();
    const uint16_t* knew = k_new + ((size_t)bl * s.Hkv + kvh) * D;
    const uint16_t* vnew = v_new + ((size_t)bl * s.Hkv + kvh) * D;

    // B operand of S^T: query head c (zero for the padding heads), 8 dims of the lane's quarter per k-step
    bf16x8 qf[KSTEPS];
    {
        const bool hv = c < G;
        const uint16_t* qp = q + ((size_t)bl * s.H + kvh * G + (hv ? c : 0)) * D + qq * 8;
#pragma unroll
        for (int ks = 0; ks < KSTEPS; ++ks) {
            u32x4 z = {0u, 0u, 0u, 0u};
            qf[ks] = as_bf16x8(hv ? load16(qp + ks * 32) : z);
        }
    }

    const int per = (len + nsplit - 1) / nsplit;
    const int t0 = min(split * per, len), t1 = min(t0 + per, len);
    const int nblk = (t1 - t0 + 15) >> 4;
    const int wblk = (nblk + 3) >> 2;  // blocks per wave, uniform over the workgroup

    float m_run = kNegInf, l_run = 0.f;
    f32x4 o[2 * NB2];
#pragma unroll
    for (int nb = 0; nb < 2 * NB2; ++nb) o[nb] = f32x4{0.f, 0.f, 0.f, 0.f};
    char* vst = smem + wave * 16 * VROWB;
    char* kst = smem + (4 + wave) * 16 * VROWB;

    // loads of the block at token n0: its K and V rows, 16 lanes per row; rows past t1
    // (and the step's own token) read the fresh k_new / v_new row, so every load is issued
    auto settle_qf = [&]() {
#pragma unroll
        for (int ks = 0; ks < KSTEPS; ++ks) settle(qf[ks]);
    };
    auto issue = [&](u32x4 (&kr)[VLOADS], u32x4 (&vr)[VLOADS], int n0) {
#pragma unroll
        for (int i = 0; i < VLOADS; ++i) {
            const int ch = i * 64 + lane;
            const int n = n0 + ch / VCH;
            const bool fresh = n >= len - 1 || n >= t1;
            const size_t r = fresh ? 0 : rows.row(n);
            kr[i] = load16_stream((fresh ? knew : kc + r) + (ch % VCH) * 8);
            vr[i] = load16_stream((fresh ? vnew : vc + r) + (ch % VCH) * 8);
        }
    };
    // rows into the wave's LDS stages, then S^T from the staged K (lane: row c, its k-step columns)
    auto stage = [&](const u32x4 (&kr)[VLOADS], const u32x4 (&vr)[VLOADS]) {
        // the stages are free: this wave's reads of the previous block were issued before
        asm volatile("" ::: "memory");
#pragma unroll
        for (int i = 0; i < VLOADS; ++i) {
            const int ch = i * 64 + lane;
            store16(vst + (ch / VCH) * VROWB + (ch % VCH) * 16, vr[i]);
            store16(kst + (ch / VCH) * VROWB + (ch % VCH) * 16, kr[i]);
        }
        asm volatile("" ::: "memory");
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < KSTEPS; ++ks)
            acc = mfma16x16x32(as_bf16x8(*reinterpret_cast<const u32x4*>(kst + c * VROWB + (ks * 32 + qq * 8) * 2)),
                               qf[ks], acc);
        return acc;
    };
    auto consume = [&](f32x4 acc, int n0) {
        float z[4], mb = kNegInf;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            z[j] = n0 + 4 * qq + j < t1 ? acc[j] * s.scale2 : kNegInf;
            mb = fmaxf(mb, z[j]);
        }
        mb = max_xor32(max_xor16(mb));
        const float m_new = fmaxf(m_run, mb);
        if (__builtin_amdgcn_ballot_w64(m_new > m_run) != 0) {  // some head's max grew (uniform branch)
            const float sc = m_new == kNegInf ? 1.f : fast_exp2(m_run - m_new);
            l_run *= sc;
            float scr[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) scr[j] = __shfl(sc, 4 * qq + j, 64);  // output row 4*qq + j's head
#pragma unroll
            for (int nb = 0; nb < 2 * NB2; ++nb)
#pragma unroll
                for (int j = 0; j < 4; ++j) o[nb][j] *= scr[j];
            m_run = m_new;
        }
        const float mu = m_run == kNegInf ? 0.f : m_run;
        bf16x4 ph, pl;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float p = fast_exp2(z[j] - mu);
            l_run += p;
            ph[j] = (__bf16)p;
            pl[j] = (__bf16)(p - (float)ph[j]);
        }
        asm volatile("" ::: "memory");
        // B operand: tokens 4*qq .. +3 of dims 32*nb2 + 2c (even block) and + 1 (odd block)
#pragma unroll
        for (int nb2 = 0; nb2 < NB2; ++nb2) {
            uint32_t w[4];
#pragma unroll
            for (int i = 0; i < 4; ++i)
                w[i] = *reinterpret_cast<const uint32_t*>(vst + (4 * qq + i) * VROWB + (32 * nb2 + 2 * c) * 2);
            typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
            const u32x2 ev = {(w[0] & 0xFFFFu) | (w[1] << 16), (w[2] & 0xFFFFu) | (w[3] << 16)};
            const u32x2 od = {(w[0] >> 16) | (w[1] & 0xFFFF0000u), (w[2] >> 16) | (w[3] & 0xFFFF0000u)};
            const bf16x4 be = __builtin_bit_cast(bf16x4, ev), bo = __builtin_bit_cast(bf16x4, od);
            o[2 * nb2] = mfma16x16x16(ph, be, o[2 * nb2]);
            o[2 * nb2] = mfma16x16x16(pl, be, o[2 * nb2]);
            o[2 * nb2 + 1] = mfma16x16x16(ph, bo, o[2 * nb2 + 1]);
            o[2 * nb2 + 1] = mfma16x16x16(pl, bo, o[2 * nb2 + 1]);
        }
    };

    u32x4 ka[VLOADS], va[VLOADS];
    int n0 = t0 + 16 * wave;  // this wave's blocks: wave, wave + 4, ... of the split
    issue(ka, va, n0);
    settle_qf();
    for (int bi = 0; bi < wblk; ++bi) {
        const f32x4 acc = stage(ka, va);
        issue(ka, va, n0 + 64);
        consume(acc, n0);
        n0 += 64;
    }

    // the step's token into its cache slot (this launch reads it from k_new / v_new)
    if (split == 0 && tid < VCH) {
        const size_t r = rows.row(bsz + st);
        store16(kc + r + tid * 8, load16(knew + tid * 8));
        store16(vc + r + tid * 8, load16(vnew + tid * 8));
    }
    // the four lane quarters summed different tokens of each head
    l_run = sum_xor32(sum_xor16(l_run));
    __syncthreads();  // every wave is done with its stage: the merge reuses it
    float* wm = reinterpret_cast<float*>(smem);  // [4][GMAX]
    float* wl = wm + 4 * GMAX;                   // [4][GMAX]
    float* wacc = wl + 4 * GMAX;                 // [4][GMAX][D]
    if (qq == 0 && c < G) {
        wm[wave * GMAX + c] = m_run;
        wl[wave * GMAX + c] = l_run;
    }
#pragma unroll
    for (int nb2 = 0; nb2 < NB2; ++nb2)
#pragma unroll
        for (int e = 0; e < 2; ++e)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int h = 4 * qq + j;
                if (h < G) wacc[(wave * GMAX + h) * D + 32 * nb2 + 2 * c + e] = o[2 * nb2 + e][j];
            }
    __syncthreads();
    for (int x = tid; x < G * D; x += kThreads) {
        const int h = x / D, dd = x % D;
        float M = kNegInf;
#pragma unroll
        for (int w = 0; w < 4; ++w) M = fmaxf(M, wm[w * GMAX + h]);
        float num = 0.f, den = 0.f;
        if (M != kNegInf) {
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                const float sc = fast_exp2(wm[w * GMAX + h] - M);
                num += sc * wacc[(w * GMAX + h) * D + dd];
                den += sc * wl[w * GMAX + h];
            }
        }
        const size_t bh = (size_t)bl * s.H + kvh * G + h;
        if (!SPLIT || nsplit == 1) {
            out[bh * D + dd] = num / den;
        } else {
            float* p = ws_part + (bh * sp.most + split) * (size_t)(D + 2);
            store_shared(p + 2 + dd, num);
            if (dd == 0) {
                store_shared(p, M);
                store_shared(p + 1, den);
            }
        }
    }
    if constexpr (SPLIT) {
        if (nsplit > 1)
            combine_splits<D, GMAX>(sp, slot, split, (size_t)bl * s.H + kvh * G, G, nsplit, ws_part, out);
    }
}

size_t partial_floats(const Shape& s, int nsplit) {
    return nsplit > 1 ? (size_t)s.B * s.L * s.H * nsplit * (s.D + 2) : 0;
}

// The call's splits: how units are split and dealt out, its marks (behind the partials, 8-byte aligned)
// and its number.
Splits call_splits(const Shape& s, float* ws_part, int nsplit) {
    if (nsplit <= 1) return Splits{nullptr, 0, 1, 1, 1, 1};
    static std::atomic<unsigned long long> next{
        (unsigned long long)std::chrono::steady_clock::now().time_since_epoch().count() * 0x9E3779B97F4A7C15ull};
    const int units = s.B * s.L * s.Hkv;  // at most 512, for a split
    unsigned long long call;
    do call = next.fetch_add(1, std::memory_order_relaxed); while (call == 0);
    const uintptr_t end = reinterpret_cast<uintptr_t>(ws_part + partial_floats(s, nsplit));
    return Splits{reinterpret_cast<unsigned long long*>((end + 7) / 8 * 8), call, nsplit,
                  std::min(std::max(kCUs / units, 1), nsplit),
                  // more units than CUs are even enough without the shorter splits (400 units of 1000 rows: 35 us
                  // against 44 in two splits)
                  units <= kCUs ? 512 : 1024, kCUs / nsplit};
}

template <int D, class Rows>
hipError_t launch_decode_d(const Shape& s, const Rows& rows, size_t lds_bytes, uint16_t* kc, uint16_t* vc,
                           const int32_t* budgets, int32_t reserve, int32_t step, const int32_t* steps,
                           const uint16_t* q, const uint16_t* k_new, const uint16_t* v_new, float* out, float* ws_part,
                           int nsplit, const int32_t* unit_order, hipStream_t st) {
    const Splits sp = call_splits(s, ws_part, nsplit);
    const long long units = (long long)s.B * s.L * s.Hkv;
    const dim3 grid((unsigned)(nsplit > 1 ? (units + sp.span - 1) / sp.span * kCUs : units)), block(kThreads);
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, grid, block, lds_bytes, st, s, rows, kc, vc, budgets, reserve, step, steps, q, k_new,
                           v_new, out, ws_part, sp, unit_order);
    };
    if (nsplit > 1) {
        if (s.G <= 1) launch(decode_kernel<D, 1, Rows, true>);
        else if (s.G < kMfmaMinGroup) launch(decode_kernel<D, 2, Rows, true>);
        else if (s.G <= 4) launch(decode_mfma_kernel<D, 4, Rows, true>);
        else if (s.G <= 8) launch(decode_mfma_kernel<D, 8, Rows, true>);
        else launch(decode_mfma_kernel<D, 16, Rows, true>);
    } else {
        if (s.G <= 1) launch(decode_kernel<D, 1, Rows, false>);
        else if (s.G < kMfmaMinGroup) launch(decode_kernel<D, 2, Rows, false>);
        else if (s.G <= 4) launch(decode_mfma_kernel<D, 4, Rows, false>);
        else if (s.G <= 8) launch(decode_mfma_kernel<D, 8, Rows, false>);
        else launch(decode_mfma_kernel<D, 16, Rows, false>);
    }
    return hipGetLastError();
}

}  // namespace

// Split partials of decode for callers that cannot allocate (tgvkv_decode_attn_noalloc):
// one buffer per GPU, living as long as the process.  Host code must not pass the array's
// name to a kernel (it is a host-side stand-in there); decode_scratch() gives its device
// address, looked up once per device with that device current.
static __device__ __align__(256) float scratch[kDecodeScratchBytes / sizeof(float)];
// every shape that is split fits: 16 query heads at most (decode_mfma_kernel), head_dim 128
static_assert(kMaxSplitGroups * (16 * (128 + 2) * sizeof(float) + sizeof(unsigned long long)) + 256 <= kDecodeScratchBytes,
              "split partials and marks in the static buffer");

hipError_t decode_scratch(float** ptr) {
    constexpr int kMaxDevices = 64;
    static std::mutex mu;
    static float* addr[kMaxDevices] = {};
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    if (addr[dev] == nullptr) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        addr[dev] = static_cast<float*>(p);
    }
    *ptr = addr[dev];
    return hipSuccess;
}

int decode_splits(const Shape& s) {
    const long long units = (long long)s.B * s.L * s.Hkv;
    if (units <= 0) return 1;
    // most workgroups per unit: about 1024 in all, 4 per CU; a unit takes as many of them as its rows are
    // worth (unit_splits), at least as many as fit one per CU: a partial costs its trip through memory and
    // the combination about 4 us at the end, and one workgroup's waves already keep a CU's share of the
    // stream in flight.  Against as many splits as workgroups for every unit, of even lengths, per step: 132
    // units of 300 rows 9.0 against 12.8 us, 112 units of 1000 rows 14.2 against 16.0; 32 units (8
    // splits either way) 7.7.
    long long n = kMaxSplitGroups / units;
    if (n < 1) n = 1;
    if (n > kMaxSplits) n = kMaxSplits;
    return (int)n;
}

size_t decode_workspace(const Shape& s) {
    const int n = decode_splits(s);
    return n <= 1 ? 0 : sizeof(float) * partial_floats(s, n) + 8 + sizeof(unsigned long long) * (size_t)s.B * s.L * s.Hkv * n;
}

hipError_t launch_decode(const Shape& s, uint16_t* kc, uint16_t* vc, const int32_t* budgets, const int64_t* seg_off,
                         int32_t reserve, int32_t step, const uint16_t* q, const uint16_t* k_new, const uint16_t* v_new,
                         float* out, float* ws_part, const int32_t* unit_order, hipStream_t st) {
    if ((long long)s.B * s.L == 0) return hipSuccess;
    const int nsplit = decode_splits(s);
    if (s.D == 128) {
        ContigRows<128> rows{seg_off, reserve, 0};
        return launch_decode_d<128>(s, rows, 0, kc, vc, budgets, reserve, step, nullptr, q, k_new, v_new, out,
                                    ws_part, nsplit, unit_order, st);
    }
    ContigRows<64> rows{seg_off, reserve, 0};
    return launch_decode_d<64>(s, rows, 0, kc, vc, budgets, reserve, step, nullptr, q, k_new, v_new, out, ws_part,
                               nsplit, unit_order, st);
}

hipError_t launch_decode_paged(const Shape& s, uint16_t* k_pool, uint16_t* v_pool, int64_t n_pages,
                               const int32_t* block_table, int32_t max_pages, int32_t page_shift,
                               const int32_t* budgets, int32_t reserve, const int32_t* steps, const uint16_t* q,
                               const uint16_t* k_new, const uint16_t* v_new, float* out, float* ws_part,
                               const int32_t* unit_order, hipStream_t st) {
    if ((long long)s.B * s.L == 0) return hipSuccess;
    const int nsplit = decode_splits(s);
    const size_t lds = PagedRows<128>::lds_bytes(max_pages);
    const int np = (int)std::min<int64_t>(n_pages, INT32_MAX);
    if (s.D == 128) {
        PagedRows<128> rows{block_table, max_pages, page_shift, np, 0, 0, nullptr};
        return launch_decode_d<128>(s, rows, lds, k_pool, v_pool, budgets, reserve, 0, steps, q, k_new, v_new, out,
                                    ws_part, nsplit, unit_order, st);
    }
    PagedRows<64> rows{block_table, max_pages, page_shift, np, 0, 0, nullptr};
    return launch_decode_d<64>(s, rows, lds, k_pool, v_pool, budgets, reserve, 0, steps, q, k_new, v_new, out,
                               ws_part, nsplit, unit_order, st);
}

}  // namespace tgvkv
