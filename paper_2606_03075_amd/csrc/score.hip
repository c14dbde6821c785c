// TWR / TVB scoring, one kernel per phase (gfx950).
//
// The method reads only the rows of the causal softmax A = softmax(tau Q K^T + M)
// (Sec. 3.1, Eq. (2)) whose queries are text tokens.  Those rows are recomputed
// here from the cached keys, because a fused prefill attention kernel does not
// return probabilities.  Two sweeps over K are unavoidable: the text-weighted
// vision scores (Eq. (8)) need each row's final normaliser and the weights w~
// (Eq. (7)), which depend on every head of the layer.
//
//   score_stats   sweep 1: question rows x all visible keys -> row log-sum-exp
//                 and vision mass, online (one K read);
//   score_stats_text  sweep 1 followed by the unit's text pass in the same
//                 workgroup, when one workgroup holds all of a unit's question rows;
//   score_text    text rows x text keys: system-row normalisers, then the
//                 text->text probabilities' column sums per head (Eq. (9)); with few units
//                 sweep 1's shares of the keys have workgroups of their own, and this merges
//                 their statistics (score_stats_merge does when these are asked for alone);
//   score_fin     head means -> s^T, w, w~ (Eq. (7), (9)) and the layer's
//                 text->vision mass (Eq. (5)-(6));
//   score_vision  sweep 2: question rows x vision keys, p = exp(z - lse),
//                 column sums weighted by w~ (Eq. (8));
//   score_vis_reduce  deterministic sum of the per-(KV head, row group) partials; when
//                 the caller gives the rows' normalisers (from its prefill) and sweep 1 is
//                 skipped, the vision sweep also yields each row's vision mass, so K is read
//                 once, and this launch forms the layers' TV masses from them.
//
// These kernels serve phase-by-phase calls (and the vision pass restricted to
// layers whose budget reaches past the text).
#include <algorithm>
#include <climits>
#include <map>
#include <mutex>
#include <tuple>
#include <type_traits>

#include "score_core.h"

namespace tgvkv {
namespace {

using namespace core;

// Partial row statistics of a sweep whose keys are summed in nsplit shares, of ks key parts each:
// [3][ks][nsplit][rows] (reference max in base-2 units, sum, vision sum), rows = B*L*H*N_q.  merge_row adds
// a row's shares in share order, then its key parts, and gives its normaliser (natural log) and vision mass.
__device__ __forceinline__ void merge_row(const float* ws_stat, size_t rows, int nsplit, int ks, size_t r,
                                          float& ln, float& vm) {
    const size_t plane = rows * nsplit * ks;
    float m = kNegInf, l = 0.f, v = 0.f;
    for (int kp = 0; kp < ks; ++kp) {
        const float* w = ws_stat + (size_t)kp * nsplit * rows + r;
        float pm = w[0], pl = w[plane], pv = w[2 * plane];
        constexpr int U = 6;  // shares' loads in flight at once
        for (int s0 = 1; s0 < nsplit; s0 += U) {
            float a[U][3];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const size_t x = min(s0 + u, nsplit - 1) * rows;
                a[u][0] = w[x];
                a[u][1] = w[plane + x];
                a[u][2] = w[2 * plane + x];
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (s0 + u < nsplit) merge_shares(pm, pl, pv, a[u][0], a[u][1], a[u][2]);
        }
        if (kp == 0) {
            m = pm;
            l = pl;
            v = pv;
        } else {
            merge_shares(m, l, v, pm, pl, pv);
        }
    }
    ln = (m + log2f(l)) * kLn2;
    vm = v / l;
}

// Keys of share sp of a unit, a multiple of the tile, and its partial statistics for the row group that
// starts at block rb0.
template <int NSLOT, int KS>
__device__ __forceinline__ void write_share(const Shape& s, int bl, int kvh, int rb0, int sp, int nsplit,
                                            const int (&qrow)[NSLOT], const float (&m)[NSLOT],
                                            const float (&lsum)[NSLOT], const float (&vsum)[NSLOT], float* ws_stat) {
    constexpr int RSETS = 4 / KS;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int rs = wave % RSETS, kp = wave / RSETS;
    const int QB = (s.Nq + 15) >> 4, NB = s.G * QB;
    if (lane >= 16) return;
    const size_t rows = (size_t)s.B * s.L * s.H * s.Nq;
#pragma unroll
    for (int sl = 0; sl < NSLOT; ++sl) {
        const int rb = slot_block<RSETS>(rb0, rs, sl);
        const int qi = qrow[sl];
        if (rb < NB && qi < s.Nq) {
            float* w = ws_stat + (kp * nsplit + sp) * rows + ((size_t)bl * s.H + kvh * s.G + rb / QB) * s.Nq + qi;
            w[0] = m[sl];
            w[rows * nsplit * KS] = lsum[sl];
            w[2 * rows * nsplit * KS] = vsum[sl];
        }
    }
}

// Sweep 1 of one row group of a unit: of one of its nsplit shares of `per` key tiles, whose statistics the
// text pass or score_stats_merge merges, or (nsplit 1) of all its keys, with SHARES in shares of `per` tiles.
template <int D, int NSLOT, int KS, bool SHARES>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(NSLOT >= 6 ? 2 : NSLOT == 3 ? 3 : 1))) void score_stats_kernel(Shape s, int rowgroups,
                                                               const uint16_t* __restrict__ q_text,
                                                               const uint16_t* __restrict__ k,
                                                               float* __restrict__ lse,
                                                               float* __restrict__ ws_vm, int nsplit, int per,
                                                               float* __restrict__ ws_stat) {
    constexpr int RSETS = 4 / KS;
    __shared__ __attribute__((aligned(16))) char tiles[2][Geo<D>::TILE_BYTES];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int rs = wave % RSETS, kp = wave / RSETS;
    int bid = blockIdx.x;
    const int sp = bid % nsplit;
    bid /= nsplit;
    const int rg = bid % rowgroups;
    bid /= rowgroups;
    const int kvh = bid % s.Hkv;
    const int bl = bid / s.Hkv;
    const int QB = (s.Nq + 15) >> 4;
    const int NB = s.G * QB;
    const int rb0 = rg * RSETS * NSLOT;

    bf16x8 qf[NSLOT][Geo<D>::KSTEPS];
    int qrow[NSLOT];
    load_qrows<D, NSLOT, KS>(s, q_text, bl, kvh, rb0, qf, qrow);
    const uint16_t* kbase = k + ((size_t)bl * s.Hkv + kvh) * (size_t)s.N * D;
    const int kbeg = sp * per * kTile, kend = min(kbeg + per * kTile, s.N);
    float m[NSLOT], lsum[NSLOT], vsum[NSLOT];
    if constexpr (SHARES)
        stats_sweep<D, NSLOT, KS, true>(s, kbase, 0, s.N, qf, qrow, tiles, m, lsum, vsum, per);
    else
        stats_sweep<D, NSLOT, KS>(s, kbase, kbeg, kend, qf, qrow, tiles, m, lsum, vsum, 0, nsplit > 1);
    if (!SHARES && nsplit > 1) {
        write_share<NSLOT, KS>(s, bl, kvh, rb0, sp, nsplit, qrow, m, lsum, vsum, ws_stat);
    } else if (kp == 0 && lane < 16) {
#pragma unroll
        for (int sl = 0; sl < NSLOT; ++sl) {
            const int rb = slot_block<RSETS>(rb0, rs, sl);
            const int qi = qrow[sl];
            if (rb < NB && qi < s.Nq) {
                const size_t head = (size_t)bl * s.H + kvh * s.G + rb / QB;
                lse[head * s.Nt + s.Ns + qi] = (m[sl] + log2f(lsum[sl])) * kLn2;
                ws_vm[head * s.Nq + qi] = vsum[sl] / lsum[sl];
            }
        }
    }
}

// Normalisers and vision masses from the shares' statistics, one thread per question row (for
// calls that ask for the statistics alone; the text pass merges them itself).
__global__ __launch_bounds__(kThreads) void score_stats_merge_kernel(Shape s, const float* __restrict__ ws_stat,
                                                                     int nsplit, int ks, float* __restrict__ lse,
                                                                     float* __restrict__ ws_vm) {
    const size_t rows = (size_t)s.B * s.L * s.H * s.Nq;
    const size_t r = (size_t)blockIdx.x * kThreads + threadIdx.x;
    if (r >= rows) return;
    float ln, vm;
    merge_row(ws_stat, rows, nsplit, ks, r, ln, vm);
    lse[r / s.Nq * s.Nt + s.Ns + r % s.Nq] = ln;
    ws_vm[r] = vm;
}

// Sweep 1 and the text pass of one unit in one workgroup, for shapes where one
// workgroup holds all question rows of a (sequence, layer, KV head): the text
// pass is latency-bound, so running it as each unit's sweep ends hides it behind
// the other workgroups' key streams, and the question rows' normalisers go to
// the text pass through LDS.  The row statistics are bit-identical to
// score_stats'; the text pass stages the unit's text keys in the freed tiles
// when they fit (a different summation order of the same column sums).
// Row plans whose statistics+text kernel has text mode 2 (text_pass_qregs): with three or four
// row slots per wave the sweep sets the kernel's register count, and the pass fits beside it;
// with fewer slots it would cost occupancy, with more it would spill.  With three slots (11 row
// blocks, 262 text rows of 450) 523 us against 721 us for text mode 1.
template <int NSLOT, int KS>
constexpr bool kQregsText = (NSLOT == 3 || NSLOT == 4) && KS == 1;

// With three or four row slots the kernel is held to 168 registers, 3 waves per SIMD: with text mode 2 it then spills
// 16 or 96 bytes a lane, all outside the sweep's tile loops (at its phase changes and in the text pass),
// and at the 13B stress shape (four slots) it took 6.84 ms against 7.21-7.25 ms at 2 waves per SIMD.
// QREGS: a kernel of its own for text mode 2, without the other modes' code: their calls beside the
// spills at 168 registers cost the 13B stress shape 5 %.
// SHARES: the unit's keys are summed in shares of share_tiles tiles and the text pass's columns BY_ROW, to the
// bits of score_stats on every share and score_text.
template <int D, int NSLOT, int KS, bool QREGS = false, bool SHARES = false>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(NSLOT == 3 || NSLOT == 4 ? 3 : SHARES && NSLOT == 6 && D == 128 ? 2 : 1))) void
score_stats_text_kernel(Shape s, const uint16_t* __restrict__ q_text, const uint16_t* __restrict__ k,
                        float* __restrict__ lse, float* __restrict__ ws_vm, float* __restrict__ ws_colsum,
                        float* __restrict__ ws_vmh, int text_mode, int share_tiles) {
    constexpr int RSETS = 4 / KS;
    __shared__ __attribute__((aligned(16))) char tiles[2][Geo<D>::TILE_BYTES];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int rs = wave % RSETS, kp = wave / RSETS;
    const int kvh = blockIdx.x % s.Hkv;
    const int bl = blockIdx.x / s.Hkv;
    const int QB = (s.Nq + 15) >> 4;
    const int NB = s.G * QB;
    const size_t head0 = (size_t)bl * s.H + kvh * s.G;

    bf16x8 qf[NSLOT][Geo<D>::KSTEPS];
    int qrow[NSLOT];
    load_qrows<D, NSLOT, KS>(s, q_text, bl, kvh, 0, qf, qrow);
    float m[NSLOT], lsum[NSLOT], vsum[NSLOT];
    const uint16_t* kbase = k + ((size_t)bl * s.Hkv + kvh) * (size_t)s.N * D;
    stats_sweep<D, NSLOT, KS, SHARES>(s, kbase, 0, s.N, qf, qrow, tiles, m, lsum, vsum, share_tiles);

    // [G][N_t] normalisers (base 2), then [G][N_q] vision masses: in the dynamic LDS area
    // (text mode 2, whose text pass streams keys through the tiles), else in the freed tiles
    extern __shared__ float tarea[];
    float* lse2s = QREGS ? tarea : reinterpret_cast<float*>(&tiles[0][0]);
    float* vms = lse2s + (size_t)s.G * s.Nt;
    if (kp == 0 && lane < 16) {
#pragma unroll
        for (int sl = 0; sl < NSLOT; ++sl) {
            const int rb = slot_block<RSETS>(0, rs, sl);
            const int qi = qrow[sl];
            if (rb < NB && qi < s.Nq) {
                const int g = rb / QB;
                const float ln = (m[sl] + log2f(lsum[sl])) * kLn2;
                const float vm = vsum[sl] / lsum[sl];
                lse[(head0 + g) * s.Nt + s.Ns + qi] = ln;
                ws_vm[(head0 + g) * s.Nq + qi] = vm;
                lse2s[g * s.Nt + s.Ns + qi] = ln * kLog2e;
                vms[g * s.Nq + qi] = vm;
            }
        }
    }
    __syncthreads();
    // per query head: the sum of its question rows' vision masses (one wave per head)
    for (int g = tid >> 6; g < s.G; g += kThreads / 64) {
        float a = 0.f;
        for (int qi = tid & 63; qi < s.Nq; qi += 64) a += vms[g * s.Nq + qi];
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) a += shfl_xor(a, off);
        if ((tid & 63) == 0) ws_vmh[head0 + g] = a;
    }
    if constexpr (QREGS) {
        static_assert(kQregsText<NSLOT, KS>, "row plan without text mode 2");
        // the question rows' fragments are still in registers: only text keys are loaded
        text_pass_qregs<D, NSLOT, KS>(s, bl, kvh, q_text, k, lse, qf, lse2s, vms + (size_t)s.G * s.Nq, tiles,
                                      ws_colsum);
    } else if (SHARES || text_mode == 1) {
        // the unit's text keys go into the freed tiles after the normalisers and masses
        const size_t off = ((size_t)s.G * (s.Nt + s.Nq) * sizeof(float) + 15) & ~(size_t)15;
        text_pass_lds<D, SHARES>(s, bl, kvh, 0, s.G, q_text, k, lse, lse2s, &tiles[0][0] + off,
                         2LL * Geo<D>::TILE_BYTES - (long long)off, ws_colsum);
    } else {
        text_pass<D>(s, bl, kvh, 0, s.G, q_text, k, lse, lse2s, ws_colsum);
    }
}

// The text pass of query heads g0 .. g0 + G - 1 of one unit by one workgroup.  ws_stat non-null: the question
// rows' statistics come as nsplit shares, merged here.  LDS: lse2s [G][N_t] row normalisers (base-2 units), and
// with kl_bytes > 0 the staged pass's area kl (16-byte aligned).
template <int D>
__device__ __forceinline__ void text_unit(const Shape& s, int bl, int kvh, int g0, int G,
                                          const uint16_t* __restrict__ q_text, const uint16_t* __restrict__ k,
                                          float* __restrict__ lse, float* __restrict__ ws_vm,
                                          float* __restrict__ ws_colsum, float* __restrict__ ws_vmh, bool lse_given,
                                          float* lse2s, char* kl, long long kl_bytes, const float* ws_stat, int nsplit,
                                          int ks, bool one_order) {
    const int tid = threadIdx.x;
    const size_t head0 = (size_t)bl * s.H + kvh * s.G + g0;
    if (lse_given) {
        // every text row's normaliser comes from the caller (a prefill kernel's row log-sum-exp)
        for (int x = tid; x < G * s.Nt; x += kThreads) lse2s[x] = lse[head0 * s.Nt + x] * kLog2e;
    } else {
        for (int x = tid; x < G * s.Nq; x += kThreads) {
            const int g = x / s.Nq, qi = x % s.Nq;
            float ln;
            if (ws_stat != nullptr) {
                float vm;
                merge_row(ws_stat, (size_t)s.B * s.L * s.H * s.Nq, nsplit, ks, (head0 + g) * s.Nq + qi, ln, vm);
                lse[(head0 + g) * s.Nt + s.Ns + qi] = ln;
                ws_vm[(head0 + g) * s.Nq + qi] = vm;
            } else {
                ln = lse[(head0 + g) * s.Nt + s.Ns + qi];
            }
            lse2s[g * s.Nt + s.Ns + qi] = ln * kLog2e;
        }
        __syncthreads();
        // per query head: the sum of its question rows' vision masses (one wave per head; in row
        // order when one order of sums is asked for)
        if (one_order) {
            if (tid < G) {
                float a = 0.f;
                for (int qi = 0; qi < s.Nq; ++qi) a += ws_vm[(head0 + tid) * s.Nq + qi];
                ws_vmh[head0 + tid] = a;
            }
        } else for (int g = tid >> 6; g < G; g += kThreads / 64) {
            float a = 0.f;
            for (int qi = tid & 63; qi < s.Nq; qi += 64) a += ws_vm[(head0 + g) * s.Nq + qi];
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) a += shfl_xor(a, off);
            if ((tid & 63) == 0) ws_vmh[head0 + g] = a;
        }
    }
    __syncthreads();
    if (kl_bytes > 0)
        text_pass_lds<D, true>(s, bl, kvh, g0, G, q_text, k, lse, lse2s, kl, kl_bytes, ws_colsum, lse_given);
    else
        text_pass<D>(s, bl, kvh, g0, G, q_text, k, lse, lse2s, ws_colsum, lse_given);
}

// The text pass of one unit, or with hsplit > 1 of one of its query heads (hsplit = G).
template <int D>
__global__ __launch_bounds__(kThreads) void score_text_kernel(Shape s, const uint16_t* __restrict__ q_text,
                                                              const uint16_t* __restrict__ k,
                                                              float* __restrict__ lse,
                                                              float* __restrict__ ws_vm,
                                                              float* __restrict__ ws_colsum,
                                                              float* __restrict__ ws_vmh, int lse_given, int hsplit,
                                                              long long kl_bytes, const float* __restrict__ ws_stat,
                                                              int nsplit, int ks, int one_order) {
    extern __shared__ float lse2s[];
    const int G = s.G / hsplit;  // query heads of this workgroup: g0 .. g0 + G - 1
    const int g0 = (blockIdx.x % hsplit) * G;
    const int kvh = blockIdx.x / hsplit % s.Hkv;
    const int bl = blockIdx.x / hsplit / s.Hkv;
    char* kl = reinterpret_cast<char*>(lse2s) + ((size_t)G * s.Nt * sizeof(float) + 15) / 16 * 16;
    text_unit<D>(s, bl, kvh, g0, G, q_text, k, lse, ws_vm, ws_colsum, ws_vmh, lse_given != 0, lse2s, kl, kl_bytes, ws_stat,
                 nsplit, ks, one_order != 0);
}

// One wave per (unit, query head, 16-key block) of the text->text column sums, when
// every text row's normaliser is given.
template <int D>
__global__ __launch_bounds__(64) void score_text_cols_kernel(Shape s, const uint16_t* __restrict__ q_text,
                                                             const uint16_t* __restrict__ k,
                                                             const float* __restrict__ lse,
                                                             float* __restrict__ ws_colsum) {
    const int TB = (s.Nt + 15) >> 4;
    long long item = blockIdx.x;
    const int kb = (int)(item % TB);
    item /= TB;
    const int g = (int)(item % s.G);
    item /= s.G;
    const int kvh = (int)(item % s.Hkv);
    const int bl = (int)(item / s.Hkv);
    text_cols_item<D>(s, bl, kvh, g, kb, q_text, k, lse, ws_colsum);
}

__global__ __launch_bounds__(kThreads) void score_fin_kernel(Shape s, const float* __restrict__ ws_colsum,
                                                             const float* __restrict__ ws_vmh,
                                                             float* __restrict__ s_txt,
                                                             float* __restrict__ w_txt,
                                                             float* __restrict__ tv_mass, int with_mass) {
    __shared__ float red[kThreads];
    finalize_group(s, (int)(blockIdx.x / s.ngroups), (int)(blockIdx.x % s.ngroups), ws_colsum, ws_vmh, s_txt, w_txt,
                   tv_mass, red, with_mass != 0);
}

// How the vision sweep's workgroups are dealt out: each (unit, row group) has vsplit shares
// of its vision keys; workgroup b < nfull takes share b whole, and the shares after those are
// each cut into `pieces` workgroups.  The cut shares are the last ones dispatched: they would
// otherwise run as a partial last round whose few workgroups, one or two key tiles in flight
// each, cannot keep HBM busy (at llavanext 4096 units over 768 resident workgroups leave 256
// for a sixth round).
struct VisionDeal {
    int vsplit;
    long long nfull;
    int pieces;
};

template <int D, int NSLOT, int KS, bool MASS>
__global__ __launch_bounds__(kThreads) void score_vision_kernel(Shape s, int rowgroups,
                                                                const uint16_t* __restrict__ q_text,
                                                                const uint16_t* __restrict__ k,
                                                                const float* __restrict__ lse,
                                                                const float* __restrict__ w_txt,
                                                                const int32_t* __restrict__ budgets,
                                                                int vis_threshold,
                                                                float* __restrict__ ws_part,
                                                                float* __restrict__ ws_vm, int out_tiles,
                                                                VisionDeal deal) {
    constexpr int RSETS = 4 / KS;
    __shared__ __attribute__((aligned(16))) char tiles[2][Geo<D>::TILE_BYTES];
    __shared__ float red[2][RSETS][kTile];
    extern __shared__ float obuf[];  // out_tiles * kTile scores
    const int vsplit = deal.vsplit;
    long long sh = blockIdx.x;  // this workgroup's share of the vision keys, and its piece of it
    int piece = 0, npieces = 1;
    if (sh >= deal.nfull) {
        const long long j = sh - deal.nfull;
        sh = deal.nfull + j / deal.pieces;
        piece = (int)(j % deal.pieces);
        npieces = deal.pieces;
    }
    const int sp = (int)(sh % vsplit);
    int bid = (int)(sh / vsplit);
    const int rg = bid % rowgroups;
    bid /= rowgroups;
    const int kvh = bid % s.Hkv;
    const int bl = bid / s.Hkv;
    const int QB = (s.Nq + 15) >> 4;
    const int NB = s.G * QB;
    const int rb0 = rg * RSETS * NSLOT;

    // a layer whose budget leaves no room for vision tokens needs no scores: its workgroups
    // leave before loading anything (at the 13B stress shape with i.i.d. text queries every
    // layer is such a layer, and loading the rows first cost 0.27 ms of a launch that computes
    // nothing)
    if (budgets != nullptr && budgets[bl] <= vis_threshold) return;
    bf16x8 qf[NSLOT][Geo<D>::KSTEPS];
    int qrow[NSLOT];
    load_qrows<D, NSLOT, KS, false>(s, q_text, bl, kvh, rb0, qf, qrow);
    float lse2[NSLOT][4], coef[NSLOT][4];
    load_row_coefs<NSLOT, KS, false>(s, bl, kvh, rb0, lse, w_txt, lse2, coef);
    settle_qrows<D, NSLOT>(qf);
#pragma unroll
    for (int sl = 0; sl < NSLOT; ++sl)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            settle(lse2[sl][j]);
            settle(coef[sl][j]);
        }
    const uint16_t* kvis = k + (((size_t)bl * s.Hkv + kvh) * (size_t)s.N + s.Ns) * D;
    float* out = ws_part + (((size_t)bl * s.Hkv + kvh) * rowgroups + rg) * (size_t)s.Nv;
    float rsum[NSLOT][4];
    // every key's score is a sum over this workgroup's rows only, so the keys split freely
    const int ntv = (s.Nv + kTile - 1) / kTile;
    const int per_t = (ntv + vsplit - 1) / vsplit;
    const int t0 = min(sp * per_t, ntv), t1 = min(t0 + per_t, ntv);
    const int per_p = (t1 - t0 + npieces - 1) / npieces;
    const int p0 = min(t0 + piece * per_p, t1), p1 = min(p0 + per_p, t1);
    const int vbeg = min(p0 * kTile, s.Nv), vend = min(p1 * kTile, s.Nv);
    vision_sweep<D, NSLOT, KS, MASS>(s, kvis, vbeg, vend, qf, lse2, coef, rb0, NB, tiles, red, obuf, out_tiles, out,
                                     rsum);
    if (MASS) {
        // each row's vision mass: the sum of its probabilities over all vision keys
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
        const int rs = wave % RSETS, kp = wave / RSETS;
        if (kp == 0 && (lane & 15) == 0) {
#pragma unroll
            for (int sl = 0; sl < NSLOT; ++sl) {
                const int rb = slot_block<RSETS>(rb0, rs, sl);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int qj = (rb % QB) * 16 + (lane >> 4) * 4 + j;
                    if (rb < NB && qj < s.Nq)
                        ws_vm[((size_t)sp * s.B * s.L * s.H + (size_t)bl * s.H + kvh * s.G + rb / QB) * s.Nq + qj] =
                            rsum[sl][j];
                }
            }
        }
    }
}

// Layer TV mass (Eq. (5)-(6)) from per-row vision masses, by one workgroup: the mean over the query
// heads of the sum of their question rows' masses, i.e. one sum over the layer's H * N_q rows.  ws_vm
// holds one row-mass partial per share of the vision keys ([vsplit][B*L*H][N_q]).  The loads are
// independent, eight in flight a thread; a thread per head, walking its rows one load after another,
// took 10-20 us in a launch of its own.
__device__ void layer_mass(const Shape& s, int bl, const float* __restrict__ ws_vm, float* __restrict__ tv_mass,
                           int vsplit) {
    __shared__ float wsum[kThreads / 64];
    const int n = s.H * s.Nq;
    const size_t share = (size_t)s.B * s.L * n;
    float a[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    if (s.Nv > 0) {  // with no vision keys the vision sweep does not run and every mass is 0
        for (int sp = 0; sp < vsplit; ++sp) {
            const float* vm = ws_vm + sp * share + (size_t)bl * n;
            int x = threadIdx.x;
            for (; x + 7 * kThreads < n; x += 8 * kThreads) {
#pragma unroll
                for (int u = 0; u < 8; ++u) a[u] += vm[x + u * kThreads];
            }
#pragma unroll
            for (int u = 0; u < 7; ++u)
                if (x + u * kThreads < n) a[u] += vm[x + u * kThreads];
        }
    }
    float t = ((a[0] + a[1]) + (a[2] + a[3])) + ((a[4] + a[5]) + (a[6] + a[7]));
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) t += shfl_xor(t, off);
    if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = t;
    __syncthreads();
    if (threadIdx.x == 0) {
        float m = 0.f;
#pragma unroll
        for (int w = 0; w < kThreads / 64; ++w) m += wsum[w];
        tv_mass[bl] = m / (float)s.H;
    }
}

// Sums the (KV head, row group) partials of every vision key; with ws_vm (row masses collected by
// the sweep) the workgroups past the keys' (blockIdx.x == nx) form the layers' TV masses.
__global__ __launch_bounds__(kThreads) void score_vis_reduce_kernel(Shape s, int rowgroups,
                                                                    const float* __restrict__ ws_part,
                                                                    const int32_t* __restrict__ budgets,
                                                                    int vis_threshold,
                                                                    float* __restrict__ s_vis, int nx,
                                                                    const float* __restrict__ ws_vm,
                                                                    float* __restrict__ tv_mass, int vsplit) {
    const int j = blockIdx.x * kThreads + threadIdx.x;
    const int gi = blockIdx.y % s.ngroups;
    const int bl = blockIdx.y / s.ngroups;
    if (blockIdx.x == nx) {
        if (gi == 0) layer_mass(s, bl, ws_vm, tv_mass, vsplit);
        return;
    }
    if (j >= s.Nv) return;
    if (budgets != nullptr && budgets[bl] <= vis_threshold) return;
    const int kv0 = s.head_mode == 0 ? 0 : gi;
    const int kvn = s.head_mode == 0 ? s.Hkv : 1;
    // the partials of (KV head, row group) pairs are consecutive rows of n_vis: eight in flight
    const float* src = ws_part + ((size_t)bl * s.Hkv + kv0) * rowgroups * (size_t)s.Nv + j;
    const int n = kvn * rowgroups;
    float a[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    int i = 0;
    for (; i + 8 <= n; i += 8) {
#pragma unroll
        for (int u = 0; u < 8; ++u) a[u] += src[(size_t)(i + u) * s.Nv];
    }
    for (; i < n; ++i) a[0] += src[(size_t)i * s.Nv];
    s_vis[((size_t)bl * s.ngroups + gi) * s.Nv + j] = ((a[0] + a[1]) + (a[2] + a[3])) + ((a[4] + a[5]) + (a[6] + a[7]));
}

#define TGVKV_ROWPLAN_DISPATCH(KERNEL, D, rp, ...)                                                \
    do {                                                                                          \
        if (rp.ks == 4) hipLaunchKernelGGL((KERNEL<D, 1, 4>), __VA_ARGS__);                       \
        else if (rp.ks == 2 && rp.nslot == 1) hipLaunchKernelGGL((KERNEL<D, 1, 2>), __VA_ARGS__); \
        else if (rp.ks == 2) hipLaunchKernelGGL((KERNEL<D, 2, 2>), __VA_ARGS__);                  \
        else if (rp.nslot == 1) hipLaunchKernelGGL((KERNEL<D, 1, 1>), __VA_ARGS__);               \
        else if (rp.nslot == 2) hipLaunchKernelGGL((KERNEL<D, 2, 1>), __VA_ARGS__);               \
        else if (rp.nslot == 3) hipLaunchKernelGGL((KERNEL<D, 3, 1>), __VA_ARGS__);               \
        else if (rp.nslot == 4) hipLaunchKernelGGL((KERNEL<D, 4, 1>), __VA_ARGS__);               \
        else if (rp.nslot == 5) hipLaunchKernelGGL((KERNEL<D, 5, 1>), __VA_ARGS__);               \
        else hipLaunchKernelGGL((KERNEL<D, 6, 1>), __VA_ARGS__);                                  \
    } while (0)

#define TGVKV_ROWPLAN_DISPATCH_M(KERNEL, D, M, rp, ...)                                                   \
    do {                                                                                                  \
        if (rp.ks == 4) hipLaunchKernelGGL((KERNEL<D, 1, 4, M>), __VA_ARGS__);                            \
        else if (rp.ks == 2 && rp.nslot == 1) hipLaunchKernelGGL((KERNEL<D, 1, 2, M>), __VA_ARGS__);      \
        else if (rp.ks == 2) hipLaunchKernelGGL((KERNEL<D, 2, 2, M>), __VA_ARGS__);                       \
        else if (rp.nslot == 1) hipLaunchKernelGGL((KERNEL<D, 1, 1, M>), __VA_ARGS__);                    \
        else if (rp.nslot == 2) hipLaunchKernelGGL((KERNEL<D, 2, 1, M>), __VA_ARGS__);                    \
        else if (rp.nslot == 3) hipLaunchKernelGGL((KERNEL<D, 3, 1, M>), __VA_ARGS__);                    \
        else if (rp.nslot == 4) hipLaunchKernelGGL((KERNEL<D, 4, 1, M>), __VA_ARGS__);                    \
        else if (rp.nslot == 5) hipLaunchKernelGGL((KERNEL<D, 5, 1, M>), __VA_ARGS__);                    \
        else hipLaunchKernelGGL((KERNEL<D, 6, 1, M>), __VA_ARGS__);                                       \
    } while (0)

template <int N>
using IC = std::integral_constant<int, N>;

// Calls f(IC<D>, IC<NSLOT>, IC<KS>, IC<MASS>) for the score_vision_kernel variant that
// launch_score_vision runs for row plan rp (NB row blocks per unit).
template <typename F>
void with_vision_variant(int d, bool mass, const RowPlan& rp, int NB, F&& f) {
    auto plan = [&](auto dd, auto m) {
        if (!decltype(m)::value && rp.nslot == 1 && rp.ks == 1) {
            if (NB == 3) f(dd, IC<2>{}, IC<2>{}, m);
            else if constexpr (!decltype(m)::value) f(dd, IC<4>{}, IC<4>{}, m);
        } else if (rp.ks == 4) f(dd, IC<1>{}, IC<4>{}, m);
        else if (rp.ks == 2 && rp.nslot == 1) f(dd, IC<1>{}, IC<2>{}, m);
        else if (rp.ks == 2) f(dd, IC<2>{}, IC<2>{}, m);
        else if (rp.nslot == 1) f(dd, IC<1>{}, IC<1>{}, m);
        else if (rp.nslot == 2) f(dd, IC<2>{}, IC<1>{}, m);
        else if (rp.nslot == 3) f(dd, IC<3>{}, IC<1>{}, m);
        else if (rp.nslot == 4) f(dd, IC<4>{}, IC<1>{}, m);
        else if (rp.nslot == 5) f(dd, IC<5>{}, IC<1>{}, m);
        else f(dd, IC<6>{}, IC<1>{}, m);
    };
    auto with_d = [&](auto m) {
        if (d == 128) plan(IC<128>{}, m);
        else plan(IC<64>{}, m);
    };
    if (mass) with_d(IC<1>{});
    else with_d(IC<0>{});
}

// Workgroups of `kernel` that the current device holds at once (its occupancy per CU times
// the CU count), asked of the runtime once per device and kernel; 0 if it cannot tell.
int resident_workgroups(const void* kernel, size_t dyn_lds) {
    static std::mutex mu;
    static std::map<std::tuple<int, const void*, size_t>, int> known;
    int dev = 0;
    if (kernel == nullptr || hipGetDevice(&dev) != hipSuccess) return 0;
    const auto key = std::make_tuple(dev, kernel, dyn_lds);
    std::lock_guard<std::mutex> lock(mu);
    const auto it = known.find(key);
    if (it != known.end()) return it->second;
    int cus = 0, per_cu = 0, n = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess &&
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, kThreads, dyn_lds) == hipSuccess)
        n = cus * per_cu;
    else
        (void)hipGetLastError();
    known[key] = n;
    return n;
}

}  // namespace

// Units (KV heads of all sequences and layers) up to which the text pass runs one workgroup per
// query head: one unit per CU, or twice as many from 12 blocks of text rows on.  Scoring with given normalisers,
// split / whole: 7 heads, 55 text rows, 336 units 109 / 102 us, 448 units 130 / 119; 83 rows, 448 units 172 / 165;
// 235 rows, 336 units 427 / 442, 448 units 529 / 525; 8 heads, 235 rows, 320 units 367 / 397.  256 units of
// 8 heads, split, against the whole pass as it was: 82 / 107 (83 rows).
long long head_split_units(const Shape& s) { return (s.Nt + 15) / 16 >= 12 ? 512 : 256; }

RowPlan plan_question_rows(const Shape& s, bool one_order) {
    const int QB = (s.Nq + 15) / 16;
    const int NB = s.G * QB;
    RowPlan rp;
    rp.one_order = one_order;
    // up to four row slots' worth of blocks: with one or two blocks the waves split each key tile
    // instead (three and four blocks: the vision sweep has launch shapes of its own)
    if (NB <= 4) {
        rp.nslot = 1;
        rp.ks = NB <= 1 ? 4 : NB == 2 ? 2 : 1;
        rp.rowgroups = NB > 0 ? 1 : 0;
        return rp;
    }
    // the fewest row groups of at most 4 waves x 6 slots (each group reads the unit's keys), all with the
    // same slots per wave, no more than it takes: an empty slot costs the statistics sweep as much as
    // a full one.  (The groups fill up in turn: 28 blocks run as 16 + 12.)  Statistics (with the text pass
    // where it is fused) and vision sweep, against slot counts of 2, 4 or 6 filled from the first group on:
    // 12 blocks 3 slots 626 + 473 against 4 slots 793 + 449 us (80 units of 40 heads, 2215 keys);
    // 20 blocks 5 slots 400 + 335 against 6 slots 426 + 374; 28 blocks in two groups of 4 slots 389 + 336
    // against 24 + 4 blocks 418 + 435; 21 blocks in two groups of 3 slots instead of one of 6: 955 + 944
    // against 841 + 794.
    rp.rowgroups = (NB + 23) / 24;
    rp.ks = 1;
    if (one_order) {
        // 2, 4 or 6 slots, filled from the first group on: the order of sums that retained sets are taken from
        rp.nslot = NB <= 8 ? 2 : NB <= 16 ? 4 : 6;
        return rp;
    }
    rp.nslot = ((NB + rp.rowgroups - 1) / rp.rowgroups + 3) / 4;
    return rp;
}

// Key tiles per share: a unit's row statistics are summed share by share, each share afresh, and the shares
// added in order (merge_shares).  The shares follow from the sequence's own shape, never from the batch, so
// that a sequence gets the same bits in any batch; whether they are dealt to workgroups of their own
// (stats_spread) is then free.  Without them one workgroup per (unit, row group) leaves most of the chip idle
// where units are few: one video of 28 layers has 112, whose statistics and text took 299 us against 123.
//
// Shares for a single sequence to fill one round of resident workgroups (4, 3, 3, 2 per CU at 1, 2, 3, 4 and more row
// slots), of four key tiles or more (six where a workgroup loads more than 16 row blocks, or one of several
// groups of them, first: 128 units of 8275 keys in that plan 168 us in shares of four, 152 of six), in rows
// of 12 key tiles or more (6 where three slots or more make each tile long and units are few).  Statistics
// and text, microseconds, whole / in shares: one layer of 32 units of 64 question rows, 1599 keys
// 31.9 / 22.4; of 4085 keys 57 / 26; one layer of 8 units of 200 rows, 4085 keys 115 / 28; of 4 units of
// 336 rows, 8275 keys 294 / 39.  A sweep of one or two slots is a stream of
// keys, and half the CUs already draw much of the bandwidth: only sequences of up to 128 units, and the
// more units the longer.  Three and four slots give up their fused text pass for the shares
// (stats_text_eligible), which costs large batches up to a tenth (512 units of 200 rows, 1599 keys: 100 / 109), so they
// have the same limit.
constexpr int kMaxShares = 32;
constexpr int kLightUnits = 128;

int share_tiles(const Shape& s, const RowPlan& rp) {
    const int tiles = (s.N + kTile - 1) / kTile;
    const long long units = (long long)s.L * s.Hkv * rp.rowgroups;  // of one sequence
    if (rp.one_order || units <= 0 || tiles < (rp.nslot <= 2 || units > kLightUnits / 2 ? 12 : 6)) return tiles;
    if (rp.rowgroups == 1 && rp.nslot <= 4 && units > kLightUnits) return tiles;
    if (rp.rowgroups == 1 && rp.nslot <= 2 && units > 5LL * tiles * rp.nslot) return tiles;
    const int per_cu = rp.nslot == 1 ? 4 : rp.nslot <= 3 ? 3 : 2;
    const int least = rp.nslot >= 5 || rp.rowgroups > 1 ? 6 : 4;
    const int n = (int)std::min<long long>(std::min<long long>(256 * per_cu / units, tiles / least), kMaxShares);
    if (n <= 1) return tiles;
    const int per = (tiles + n - 1) / n;  // the last share takes what remains
    return rp.nslot <= 2 ? (per + 1) / 2 * 2 : per;  // an even number with two tiles in flight (stats_sweep)
}

int stats_splits(const Shape& s, const RowPlan& rp) {
    const int tiles = (s.N + kTile - 1) / kTile, per = share_tiles(s, rp);
    return (tiles + per - 1) / per;
}

// Whether the shares go to workgroups of their own, and the text pass merges them; else a workgroup sweeps a
// unit's shares one after another.  Up to 256 units, one per CU (224 of six slots and 8256 keys take 317 us
// in one workgroup each, 240 spread; 448 units 409 and 426); one- and two-slot sweeps up to 128, or
// more the longer they are (128 units of 1599 keys 33.6 and 30.5, 256 units 35.8 and 38.2; 256 units of 8275 keys 115 and
// 107, 512 units 186 and 193).
bool stats_spread(const Shape& s, const RowPlan& rp) {
    if (stats_splits(s, rp) == 1) return false;
    const long long units = (long long)s.B * s.L * s.Hkv * rp.rowgroups;
    const int tiles = (s.N + kTile - 1) / kTile;
    if (rp.nslot <= 2 && rp.rowgroups == 1) return units <= std::max(128, std::min(4 * tiles * rp.nslot, 384));
    return units <= 256;
}

hipError_t launch_score_stats(const Shape& s, const RowPlan& rp, const uint16_t* q_text, const uint16_t* k,
                              float* lse, float* ws_vm, float* ws_stat, bool merge, hipStream_t st) {
    const int nsplit = stats_spread(s, rp) ? stats_splits(s, rp) : 1;
    const bool shares = nsplit == 1 && stats_splits(s, rp) > 1;  // one after another in one workgroup
    const long long nblk = (long long)s.B * s.L * s.Hkv * rp.rowgroups * nsplit;
    if (nblk == 0) return hipSuccess;
    dim3 grid((unsigned)nblk), block(kThreads);
    const int per = share_tiles(s, rp);
    auto launch = [&](auto d) {
        constexpr int D = decltype(d)::value;
        if (shares)
            TGVKV_ROWPLAN_DISPATCH_M(score_stats_kernel, D, true, rp, grid, block, 0, st, s, rp.rowgroups, q_text, k, lse, ws_vm, nsplit, per, ws_stat);
        else
            TGVKV_ROWPLAN_DISPATCH_M(score_stats_kernel, D, false, rp, grid, block, 0, st, s, rp.rowgroups, q_text, k, lse, ws_vm, nsplit, per, ws_stat);
    };
    if (s.D == 128) launch(IC<128>{});
    else launch(IC<64>{});
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || nsplit == 1 || !merge) return e;
    const long long rows = (long long)s.B * s.L * s.H * s.Nq;
    hipLaunchKernelGGL(score_stats_merge_kernel, dim3((unsigned)((rows + kThreads - 1) / kThreads)), block, 0, st, s,
                       ws_stat, nsplit, rp.ks, lse, ws_vm);
    return hipGetLastError();
}

bool stats_text_eligible(const Shape& s, const RowPlan& rp) {
    if (rp.rowgroups != 1 || s.Nt == 0 || stats_spread(s, rp)) return false;
    const long long tile_bytes = 2LL * kTile * (2 * s.D + 16);
    if (stats_splits(s, rp) > 1) {
        if (rp.nslot == 3 || rp.nslot == 4) return false;  // the text pass is the staged one (launch_score_text stages these too)
        const long long head = ((long long)s.G * (s.Nt + s.Nq) * 4 + 15) / 16 * 16;
        return s.D == 128 ? text_lds_fits<128>(s.G, s.Ns, s.Nt, tile_bytes - head)
                          : text_lds_fits<64>(s.G, s.Ns, s.Nt, tile_bytes - head);
    }
    const long long floats = (long long)s.G * (s.Nt + s.Nq);
    return floats * 4 <= tile_bytes;
}

hipError_t launch_score_stats_text(const Shape& s, const RowPlan& rp, const uint16_t* q_text, const uint16_t* k,
                                   float* lse, float* ws_vm, float* ws_colsum, float* ws_vmh, hipStream_t st) {
    const long long nblk = (long long)s.B * s.L * s.Hkv;
    if (nblk == 0) return hipSuccess;
    dim3 grid((unsigned)nblk), block(kThreads);
    if (stats_splits(s, rp) > 1) {
        const int per = share_tiles(s, rp);
        auto launch = [&](auto d) {
            constexpr int D = decltype(d)::value;
            auto go = [&](auto kernel) {
                hipLaunchKernelGGL(kernel, grid, block, 0, st, s, q_text, k, lse, ws_vm, ws_colsum, ws_vmh, 1, per);
            };
            if (rp.ks == 4) go(score_stats_text_kernel<D, 1, 4, false, true>);
            else if (rp.ks == 2) go(score_stats_text_kernel<D, 1, 2, false, true>);
            else if (rp.nslot == 1) go(score_stats_text_kernel<D, 1, 1, false, true>);
            else if (rp.nslot == 2) go(score_stats_text_kernel<D, 2, 1, false, true>);
            else if (rp.nslot == 5) go(score_stats_text_kernel<D, 5, 1, false, true>);
            else go(score_stats_text_kernel<D, 6, 1, false, true>);
        };
        if (s.D == 128) launch(IC<128>{});
        else launch(IC<64>{});
        return hipGetLastError();
    }
    // Text mode 2 (the question rows' fragments reused from the sweep, the system keys staged
    // in the tiles, the question keys streamed through them) needs the normalisers, masses and
    // column partials in a dynamic LDS area that leaves the kernel's occupancy as it is.
    // Otherwise mode 1 stages the unit's text keys (in chunks of key blocks, if need be) in
    // the freed key tiles, after the normalisers and masses, when its partials and the system
    // keys' blocks fit there; else mode 0 reads them from memory.
    const long long tile_bytes = 2LL * kTile * (2 * s.D + 16);
    const long long area = text_area_floats(s.G, s.Nt, s.Nq) * (long long)sizeof(float);
    const int occupancy = rp.nslot == 1 ? 4 : rp.nslot <= 4 ? 3 : 2;
    const bool qregs = (rp.nslot == 3 || rp.nslot == 4) && rp.ks == 1 && s.Ns <= 2 * kTile && area <= 163840 / occupancy - tile_bytes;
    const long long head = ((long long)s.G * (s.Nt + s.Nq) * 4 + 15) / 16 * 16;
    if (qregs) {
        auto launch = [&](auto d, auto ns) {
            hipLaunchKernelGGL((score_stats_text_kernel<decltype(d)::value, decltype(ns)::value, 1, true>), grid, block,
                               (size_t)area, st, s, q_text, k, lse, ws_vm, ws_colsum, ws_vmh, 2, 0);
        };
        if (s.D == 128 && rp.nslot == 3) launch(IC<128>{}, IC<3>{});
        else if (s.D == 128) launch(IC<128>{}, IC<4>{});
        else if (rp.nslot == 3) launch(IC<64>{}, IC<3>{});
        else launch(IC<64>{}, IC<4>{});
        return hipGetLastError();
    }
    if (s.D == 128) {
        const int mode = text_lds_fits<128>(s.G, s.Ns, s.Nt, tile_bytes - head) ? 1 : 0;
        TGVKV_ROWPLAN_DISPATCH(score_stats_text_kernel, 128, rp, grid, block, 0, st, s, q_text, k, lse, ws_vm,
                               ws_colsum, ws_vmh, mode, 0);
    } else {
        const int mode = text_lds_fits<64>(s.G, s.Ns, s.Nt, tile_bytes - head) ? 1 : 0;
        TGVKV_ROWPLAN_DISPATCH(score_stats_text_kernel, 64, rp, grid, block, 0, st, s, q_text, k, lse, ws_vm,
                               ws_colsum, ws_vmh, mode, 0);
    }
    return hipGetLastError();
}

hipError_t launch_score_text(const Shape& s, const RowPlan& rp, const uint16_t* q_text, const uint16_t* k, float* lse,
                             float* ws_vm, float* ws_colsum, float* ws_vmh, const float* ws_stat, bool lse_given,
                             hipStream_t st) {
    const long long nblk = (long long)s.B * s.L * s.Hkv;
    if (nblk == 0 || s.Nt == 0) return hipSuccess;
    // the unit's text keys staged in LDS (text_pass_lds; in chunks of key blocks when they do not
    // all fit beside the normalisers): against one wave per (unit, head, 16-key block) walking the row
    // blocks from global memory, at llavanext 80 -> 20 us.  Within 40 KB, four workgroups per CU, when
    // that leaves chunks of six key blocks, else within 64 KB: the pass is latency-bound, and 230 text
    // rows took 85 us in one chunk with two workgroups per CU, 60 us in two chunks with four (224 units
    // of 7 heads); 130 rows 47 and 43 us.
    const int TB = (s.Nt + 15) / 16;
    const int sys = lse_given ? 0 : s.Ns;
    auto head_bytes = [&](int G) { return ((long long)G * s.Nt * 4 + 15) / 16 * 16; };
    auto fit = [&](auto d, int G) -> long long {  // bytes of the staged pass for G heads; 0: not staged
        constexpr int D = decltype(d)::value;
        for (const long long cap : {40960LL, 65536LL}) {
            const long long k = std::min<long long>(text_part_bytes<D>(G, s.Nt) + 16LL * TB * Geo<D>::ROWB, cap - head_bytes(G));
            if (k > 0 && text_lds_fits<D>(G, sys, s.Nt, k) &&
                (cap == 65536LL || text_chunk_blocks<D>(G, s.Nt, k) >= std::min(TB, 6)))
                return k;
        }
        return 0;
    };
    auto staged_bytes = [&](int G) { return rp.one_order ? 0LL : s.D == 128 ? fit(IC<128>{}, G) : fit(IC<64>{}, G); };
    // With few units, one workgroup per query head: each stages the unit's text keys again (from
    // cache), but a unit's heads no longer follow one another in the same four waves; also where only one
    // head's partials leave room for the keys (the sums have one order either way, staged or not)
    long long kl = staged_bytes(s.G);
    int hsplit = 1;
    if (s.G > 1 && !rp.one_order && (nblk <= head_split_units(s) || kl == 0)) {
        hsplit = s.G;
        kl = staged_bytes(1);
    }
    const int G = s.G / hsplit;
    const long long head = head_bytes(G);
    const bool staged = kl > 0;
    if (lse_given && !staged) {
        const long long items = nblk * s.G * TB;
        if (s.D == 128)
            hipLaunchKernelGGL(score_text_cols_kernel<128>, dim3((unsigned)items), dim3(64), 0, st, s, q_text, k, lse,
                               ws_colsum);
        else
            hipLaunchKernelGGL(score_text_cols_kernel<64>, dim3((unsigned)items), dim3(64), 0, st, s, q_text, k, lse,
                               ws_colsum);
        return hipGetLastError();
    }
    dim3 grid((unsigned)(nblk * hsplit)), block(kThreads);
    const size_t lds = staged ? (size_t)(head + kl) : sizeof(float) * (size_t)G * s.Nt;
    const int nsplit = stats_spread(s, rp) ? stats_splits(s, rp) : 1;
    if (nsplit == 1) ws_stat = nullptr;
    if (s.D == 128)
        hipLaunchKernelGGL(score_text_kernel<128>, grid, block, lds, st, s, q_text, k, lse, ws_vm, ws_colsum, ws_vmh,
                           (int)lse_given, hsplit, kl, ws_stat, nsplit, rp.ks, (int)rp.one_order);
    else
        hipLaunchKernelGGL(score_text_kernel<64>, grid, block, lds, st, s, q_text, k, lse, ws_vm, ws_colsum, ws_vmh,
                           (int)lse_given, hsplit, kl, ws_stat, nsplit, rp.ks, (int)rp.one_order);
    return hipGetLastError();
}

hipError_t launch_score_fin(const Shape& s, const float* ws_colsum, const float* ws_vmh, float* s_txt,
                            float* w_txt, float* tv_mass, bool with_mass, hipStream_t st) {
    const long long nblk = (long long)s.B * s.L * s.ngroups;
    if (nblk == 0) return hipSuccess;
    hipLaunchKernelGGL(score_fin_kernel, dim3((unsigned)nblk), dim3(kThreads), 0, st, s, ws_colsum, ws_vmh,
                       s_txt, w_txt, tv_mass, (int)with_mass);
    return hipGetLastError();
}

// Workgroups of the vision sweep that fill a CU: 3, and 2 of the kernels whose registers allow no more, the plain
// sweep of six slots at head_dim 128 and the mass-collecting one, which keeps a sum per row as well, from three
// slots on (five at head_dim 64).  The small kernels fit more often, which measured no better (384 units
// of 5 key tiles 17 us in 2 shares, 20 in 5).
int vision_workgroups_per_cu(const Shape& s, const RowPlan& rp, bool mass) {
    const int narrow = mass ? (s.D == 128 ? 3 : 5) : s.D == 128 ? 6 : 7;  // row slots from which 2
    return rp.nslot >= narrow ? 2 : 3;
}

int vision_splits(const Shape& s, const RowPlan& rp, bool mass) {
    // With few (unit, row group) workgroups the vision keys are split over several.  Up to 384, into the number
    // of shares, each of 2 key tiles or more but the last, whose rounds of resident workgroups take least, a round
    // being the share's tiles and about two more to start and end it: one video (112 units) in 4 shares 116 us
    // against 125 us in 8 (1.75 rounds); one layer of 128 units 32 -> 24.5 us.  The count of residents matters: with 3
    // instead of 2 per CU, 128 units of 12 row blocks with given normalisers and 8192 vision keys took 123 us in 6
    // shares, 99 in 4; with 2 instead of 3, 192 units of 20 blocks 182 us in 2, 154 in 4.  Up to
    // 2048 workgroups two rounds: at the
    // Qwen2-VL shape (896 units, 2 workgroups per CU) two splits balance the last round (805 -> 740
    // us); at 4096 units a split only adds prologues.  The mass-collecting variant writes one row-mass
    // partial per share, which the reduction adds.
    const long long units = (long long)s.B * s.L * s.Hkv * rp.rowgroups;
    if (units <= 0) return 1;
    if (units > 384) return (int)std::min<long long>(std::max<long long>(2048 / units, 1), 4);
    const long long round = 256LL * vision_workgroups_per_cu(s, rp, mass);
    const int tiles = (s.Nv + kTile - 1) / kTile;
    int best = 1;
    long long least = LLONG_MAX;
    for (int n = 1; n <= std::min(tiles / 2, kMaxShares); ++n) {
        const int per = (tiles + n - 1) / n, shares = (tiles + per - 1) / per;  // no share is empty
        const long long t = (units * shares + round - 1) / round * (per + 2);
        if (t < least) {
            least = t;
            best = shares;
        }
    }
    return best;
}

hipError_t launch_score_vision(const Shape& s, const RowPlan& rp, const uint16_t* q_text, const uint16_t* k,
                               const float* lse, const float* w_txt, const int32_t* budgets,
                               int32_t vis_threshold, float* ws_part, float* ws_vm, hipStream_t st) {
    const bool mass = ws_vm != nullptr;
    const long long units = (long long)s.B * s.L * s.Hkv * rp.rowgroups;
    const int vsplit = vision_splits(s, rp, mass);
    const long long nsh = units * vsplit;
    if (nsh == 0 || s.Nv == 0) return hipSuccess;
    // a unit's scores are kept in LDS and written once at the end when they fit (no global
    // store among the key loads); otherwise in bursts of kOutTiles tiles
    const int ntiles = ((s.Nv + kTile - 1) / kTile + vsplit - 1) / vsplit;
    const int out_tiles = (!mass && ntiles * kTile * (int)sizeof(float) <= kWholeOutBytes) ? ntiles : kOutTiles;
    const size_t obytes = (size_t)out_tiles * kTile * sizeof(float);
    // the kernel variant this plan runs, and how many of its workgroups the GPU holds at once
    const int NB = s.G * ((s.Nq + 15) / 16);
    const void* fn = nullptr;
    with_vision_variant(s.D, mass, rp, NB, [&](auto d, auto ns, auto kss, auto m) {
        fn = (const void*)&score_vision_kernel<decltype(d)::value, decltype(ns)::value, decltype(kss)::value,
                                               decltype(m)::value != 0>;
    });
    // the shares that would make a partial last round are cut into pieces that fill it (each
    // piece at least 4 key tiles); the mass-collecting sweep keeps one row-mass partial per share
    VisionDeal deal{vsplit, nsh, 1};
    const int slots = mass ? 0 : resident_workgroups(fn, obytes);
    if (slots > 0 && nsh > slots && nsh % slots != 0) {
        const long long r = nsh % slots;
        const int most = std::max(ntiles / 4, 1);
        const int pieces = (int)std::min<long long>((slots + r - 1) / r, most);
        if (pieces > 1) deal = VisionDeal{vsplit, nsh - r, pieces};
    }
    const long long nblk = deal.nfull + (nsh - deal.nfull) * deal.pieces;
    dim3 grid((unsigned)nblk), block(kThreads);
    if (mass) {
        if (s.D == 128) TGVKV_ROWPLAN_DISPATCH_M(score_vision_kernel, 128, true, rp, grid, block, obytes, st, s, rp.rowgroups, q_text, k, lse, w_txt, budgets, vis_threshold, ws_part, ws_vm, out_tiles, deal);
        else TGVKV_ROWPLAN_DISPATCH_M(score_vision_kernel, 64, true, rp, grid, block, obytes, st, s, rp.rowgroups, q_text, k, lse, w_txt, budgets, vis_threshold, ws_part, ws_vm, out_tiles, deal);
    } else if (rp.nslot == 1 && rp.ks == 1 && (s.G * ((s.Nq + 15) / 16)) == 3) {
        // three 16-row blocks per unit: two slots over half of each key tile (same row groups);
        // at the LLaVA-1.5 shape 43 us against 46-48 us for the four-slot shape below
        const RowPlan r2{2, 2, rp.rowgroups, rp.one_order};
        if (s.D == 128)
            TGVKV_ROWPLAN_DISPATCH_M(score_vision_kernel, 128, false, r2, grid, block, obytes, st, s, rp.rowgroups, q_text, k, lse, w_txt, budgets, vis_threshold, ws_part, ws_vm, out_tiles, deal);
        else
            TGVKV_ROWPLAN_DISPATCH_M(score_vision_kernel, 64, false, r2, grid, block, obytes, st, s, rp.rowgroups, q_text, k, lse, w_txt, budgets, vis_threshold, ws_part, ws_vm, out_tiles, deal);
    } else if (rp.nslot == 1 && rp.ks == 1) {
        // four 16-row blocks per unit: the vision sweep runs faster with every wave holding all
        // four blocks over a quarter of each key tile (same row groups, so the same partials)
        if (s.D == 128)
            hipLaunchKernelGGL((score_vision_kernel<128, 4, 4, false>), grid, block, obytes, st, s, rp.rowgroups,
                               q_text, k, lse, w_txt, budgets, vis_threshold, ws_part, ws_vm, out_tiles, deal);
        else
            hipLaunchKernelGGL((score_vision_kernel<64, 4, 4, false>), grid, block, obytes, st, s, rp.rowgroups,
                               q_text, k, lse, w_txt, budgets, vis_threshold, ws_part, ws_vm, out_tiles, deal);
    } else {
        if (s.D == 128) TGVKV_ROWPLAN_DISPATCH_M(score_vision_kernel, 128, false, rp, grid, block, obytes, st, s, rp.rowgroups, q_text, k, lse, w_txt, budgets, vis_threshold, ws_part, ws_vm, out_tiles, deal);
        else TGVKV_ROWPLAN_DISPATCH_M(score_vision_kernel, 64, false, rp, grid, block, obytes, st, s, rp.rowgroups, q_text, k, lse, w_txt, budgets, vis_threshold, ws_part, ws_vm, out_tiles, deal);
    }
    return hipGetLastError();
}

hipError_t launch_score_vis_reduce(const Shape& s, const RowPlan& rp, const float* ws_part, const int32_t* budgets,
                                   int32_t vis_threshold, float* s_vis, const float* ws_vm, float* tv_mass,
                                   hipStream_t st) {
    const long long ny = (long long)s.B * s.L * s.ngroups;
    const bool mass = ws_vm != nullptr;
    const int nx = (s.Nv + kThreads - 1) / kThreads;
    if (ny == 0 || nx + (int)mass == 0) return hipSuccess;
    // With no question rows there are no partials (rowgroups == 0) and every score is zero.
    dim3 grid((unsigned)(nx + (int)mass), (unsigned)ny);
    hipLaunchKernelGGL(score_vis_reduce_kernel, grid, dim3(kThreads), 0, st, s, rp.rowgroups, ws_part, budgets,
                       vis_threshold, s_vis, nx, ws_vm, tv_mass, vision_splits(s, rp, true));
    return hipGetLastError();
}

}  // namespace tgvkv
