// TPR: text-prioritised retention (Sec. 3.3, Eq. (10)).
//
// One workgroup per (sequence, layer, group).  The retained set is forced
// positions first (first n_sink, last n_recent), then either the top text tokens
// by s^T (the budget does not cover the remaining text) or all text and the top
// vision tokens by s^V.  The top-k is an exact radix select on order-preserving
// 32-bit keys, which yields the k-th largest key and how many of its ties to take;
// ties go to the lower position.  The retained positions are emitted already in
// ascending order, with no sort: each wave takes a contiguous run of 64-position
// groups, wave ballots count and rank the ties and the kept positions, and the waves'
// counts, added across one barrier, give each run the rank of its first tie and the
// output slot of its first kept position.  The work is a few latency-bound rounds per
// (sequence, layer, group), and there are few such units, so long rows get 1024 threads.
// Without TPR (an ablation of Table 5) all non-forced positions compete on one scale:
// text by s^T, vision by s^V times a factor (N_t under TWR, whose weights sum to 1).
//
// Rows up to 12288 positions keep their keys in registers, in the emission's layout (a lane's
// keys are its positions of the wave's groups): each score is read once, with every load of the
// row in flight, and neither the select's passes nor the emission touch memory again.  The select
// starts at the highest bit in which the row's keys differ and takes 9 to 11 bits a pass, so scores of
// similar size spread over the bins at once (an 8-bit pass from the top puts nearly all of them in one
// or two bins, whose LDS atomics then serialise); once at most 64 keys share the k-th key's
// digits, one wave ranks them all against all.  Longer rows re-read the scores in four 8-bit
// passes.  8256 positions, 224 rows: 25.2 -> 16.2 us; 2979 positions, 128 rows: 12.7 -> 8.3 us;
// 651 positions, 32 rows: 6.5 -> 5.3 us (replayed from a graph).
#include "tgvkv_device.h"
#include "tgvkv_shape.h"

namespace tgvkv {
namespace {

constexpr int kThreads = 1024;  // of the kernel for long rows
constexpr int kWaves = kThreads / 64;
constexpr int kRegGroups = 12;  // most 64-position groups per wave kept in registers: 12288 positions by 16 waves
// Digits of the register select: two bins a thread.
constexpr int digit_bits(int waves) { return waves >= 16 ? 11 : waves >= 8 ? 10 : 9; }
enum { MODE_FORCED = 0, MODE_TEXT = 1, MODE_VIS = 2, MODE_JOINT = 3 };
constexpr uint32_t kNotCand = 0u;  // keys of candidates are >= 1 (RowCtx::key_of)

struct RowCtx {
    int N, Ns, Nv, Nt, fs, fr;  // forced = [0, fs) U [fr, N)
    int mode;
    float vscale;               // factor on s^V in the joint ranking
    const float* sv;            // s_vis row (n_vis)
    const float* st;            // s_txt row (N_t)
    __device__ bool forced(int p) const { return p < fs || p >= fr; }
    __device__ bool is_vis(int p) const { return p >= Ns && p < Ns + Nv; }
    __device__ bool cand(int p) const {
        if (mode == MODE_FORCED) return forced(p);
        if (forced(p)) return false;
        if (mode == MODE_JOINT) return true;
        return mode == MODE_VIS ? is_vis(p) : !is_vis(p);
    }
    // key of a candidate (only called when cand(p)) with score x; never kNotCand, whatever the score's bits
    // (those of a NaN that are all ones would map to 0): the select counts on as many keys as candidates.
    // The forced positions all get one key, so the ties-to-lower-position rule takes the first ones.
    __device__ uint32_t key_of(int p, float x) const {
        if (mode == MODE_FORCED) return 1u;
        if (mode == MODE_JOINT && is_vis(p)) x *= vscale;
        return max(ordered_key(x), 1u);
    }
    __device__ uint32_t key(int p) const {
        return key_of(p, is_vis(p) ? sv[p - Ns] : st[p < Ns ? p : p - Nv]);
    }
    // kept without competing (forced in the text/vision modes, all text in the vision mode)
    __device__ bool kept_outright(int p) const {
        if (mode == MODE_FORCED) return false;
        if (forced(p)) return true;
        return mode == MODE_VIS && !is_vis(p);
    }
};

// Wave 0 finds the digit d (scanning 255 down to 0) where the running count of
// larger digits first reaches kr; writes d and kr minus the count above d.
__device__ void find_digit(const int* hist, int kr, uint32_t* sel) {
    const int lane = threadIdx.x & 63;
    // lane j owns digits 255-4j .. 252-4j
    int c[4];
    int tot = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        c[i] = hist[255 - 4 * lane - i];
        tot += c[i];
    }
    int incl = tot;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int y = __shfl_up(incl, o, 64);
        if (lane >= o) incl += y;
    }
    const int excl = incl - tot;
    const unsigned long long hit = __ballot(incl >= kr);
    const int first = hit ? __ffsll((long long)hit) - 1 : 63;
    if (lane == first) {
        int above = excl, d = 252 - 4 * lane;
        for (int i = 0; i < 4; ++i) {
            if (above + c[i] >= kr) {
                d = 255 - 4 * lane - i;
                break;
            }
            above += c[i];
        }
        sel[0] = (uint32_t)d;
        sel[1] = (uint32_t)(kr - above);
    }
}

// The row's layout and mode for its budget; k: how many candidates to take, nc: how many there are.
__device__ __forceinline__ RowCtx row_ctx(const Shape& s, const float* s_vis, const float* s_txt, int bl, int gi,
                                          int bgt, int& k, int& nc) {
    RowCtx c;
    c.N = s.N;
    c.Ns = s.Ns;
    c.Nv = s.Nv;
    c.Nt = s.Nt;
    c.fs = min(s.n_sink, s.N);
    c.fr = max(s.N - s.n_recent, c.fs);
    c.vscale = s.vision_rank == 0 ? (float)s.Nt : 1.f;
    c.sv = s_vis + ((size_t)bl * s.ngroups + gi) * s.Nv;
    c.st = s_txt + ((size_t)bl * s.ngroups + gi) * s.Nt;

    // forced positions, and text positions that are not forced: [fs, min(Ns, fr)) and
    // [max(Ns + Nv, fs), fr), from the layout alone
    const int nf = c.fs + (s.N - c.fr);
    const int ntf = max(0, min(s.Ns, c.fr) - c.fs) + max(0, c.fr - max(s.Ns + s.Nv, c.fs));

    if (bgt <= nf) { c.mode = MODE_FORCED; k = bgt; }
    else if (s.joint_rank) { c.mode = MODE_JOINT; k = bgt - nf; }
    else if (bgt - nf <= ntf) { c.mode = MODE_TEXT; k = bgt - nf; }
    else { c.mode = MODE_VIS; k = bgt - nf - ntf; }
    nc = c.mode == MODE_FORCED ? nf
                 : c.mode == MODE_JOINT  ? s.N - nf
                 : c.mode == MODE_TEXT   ? ntf
                                         : s.N - nf - ntf;
    return c;
}

__global__ __launch_bounds__(kThreads) void select_long_kernel(Shape s, const float* __restrict__ s_vis,
                                                          const float* __restrict__ s_txt,
                                                          const int32_t* __restrict__ budgets,
                                                          const int64_t* __restrict__ idx_off,
                                                          int32_t* __restrict__ idx) {
    __shared__ int hist[256];
    __shared__ int wtot[kWaves][2];
    __shared__ uint32_t sel[2];
    const int tid = threadIdx.x;
    const int gi = blockIdx.x % s.ngroups;
    const int bl = blockIdx.x / s.ngroups;
    const int bgt = budgets[bl];
    int32_t* out = idx + idx_off[bl] + (int64_t)gi * bgt;

    int k, nc;
    const RowCtx c = row_ctx(s, s_vis, s_txt, bl, gi, bgt, k, nc);

    auto key_at = [&](int p) -> uint32_t { return c.cand(p) ? c.key(p) : kNotCand; };

    uint32_t thr;
    int take_ties;
    if (k <= 0) { thr = 0xFFFFFFFFu; take_ties = 0; }
    else if (k >= nc) { thr = 0u; take_ties = nc; }
    else {
        uint32_t prefix = 0u, mask = 0u;
        int kr = k;
        for (int shift = 24; shift >= 0; shift -= 8) {
            if (tid < 256) hist[tid] = 0;
            __syncthreads();
            for (int p = tid; p < s.N; p += kThreads) {
                const uint32_t key = key_at(p);
                if (key != kNotCand && (key & mask) == prefix) atomicAdd(&hist[(key >> shift) & 255u], 1);
            }
            __syncthreads();
            if (tid < 64) find_digit(hist, kr, sel);
            __syncthreads();
            prefix |= sel[0] << shift;
            mask |= 0xFFu << shift;
            kr = (int)sel[1];
        }
        thr = prefix;
        take_ties = kr;
    }

    // ordered emission.  A tie is kept while its rank among the ties (in position order) is
    // below take_ties, so the kept ties before a position are min(take_ties, ties before it).
    // Each wave owns a contiguous run of 64-position groups.  It counts its ties and its other
    // kept positions (ballots only); one barrier, and every wave adds the counts of the waves
    // before it; then it walks its groups again, ranking each group's ties and kept positions
    // by ballots, and writes the kept positions in order.
    const int lane = tid & 63, wave = tid >> 6;
    const unsigned long long below = (1ull << lane) - 1ull;
    const int ngrp = (s.N + 63) >> 6;
    const int gpw = (ngrp + kWaves - 1) / kWaves;
    const int g0 = min(wave * gpw, ngrp), g1 = min(g0 + gpw, ngrp);
    auto classify = [&](int p, bool& tie) {  // kept outright or above the threshold; tie
        tie = false;
        if (p >= s.N) return false;
        const uint32_t key = key_at(p);
        const bool outright = c.kept_outright(p);
        const bool cand = !outright && key != kNotCand && c.cand(p);
        tie = cand && key == thr;
        return outright || (cand && key > thr);
    };
    int nt = 0, nk = 0;  // uniform over the wave
    for (int gq = g0; gq < g1; ++gq) {
        bool tie;
        const bool other = classify(gq * 64 + lane, tie);
        nt += __popcll(__ballot(tie));
        nk += __popcll(__ballot(other));
    }
    if (lane == 0) {
        wtot[wave][0] = nt;
        wtot[wave][1] = nk;
    }
    __syncthreads();
    int tb = 0, ob = 0;  // ties and other kept positions before this wave's run
    for (int w = 0; w < wave; ++w) {
        tb += wtot[w][0];
        ob += wtot[w][1];
    }
    for (int gq = g0; gq < g1; ++gq) {
        const int p = gq * 64 + lane;
        bool tie;
        const bool other = classify(p, tie);
        const unsigned long long tm = __ballot(tie);
        const bool keep = other || (tie && tb + __popcll(tm & below) < take_ties);
        const unsigned long long km = __ballot(keep);
        const int pos = ob + min(take_ties, tb) + __popcll(km & below);
        if (keep && pos < bgt) out[pos] = p;
        tb += __popcll(tm);
        ob += __popcll(__ballot(other));
    }
}

// The k-th largest of a row whose keys lie in registers: thr its key, take_ties how many keys equal
// to it are taken (kNotCand marks non-candidates; 0 < k < number of candidates).
template <int WAVES, int GPW>
__device__ __forceinline__ void select_threshold(const uint32_t (&key)[GPW], int k, int* hist, uint32_t* list,
                                                 uint32_t (*wred)[2], uint32_t* sel, uint32_t& thr, int& take_ties) {
    constexpr int THREADS = 64 * WAVES, BITS = digit_bits(WAVES), BINS = 1 << BITS;
    static_assert(BINS == 2 * THREADS, "two bins a thread");
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // smallest and largest candidate key
    uint32_t lo = 0xFFFFFFFFu, hi = 0u;
#pragma unroll
    for (int i = 0; i < GPW; ++i) {
        lo = min(lo, key[i] != kNotCand ? key[i] : 0xFFFFFFFFu);
        hi = max(hi, key[i]);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        lo = min(lo, shfl_xor(lo, o));
        hi = max(hi, shfl_xor(hi, o));
    }
    if (lane == 0) {
        wred[wave][0] = lo;
        wred[wave][1] = hi;
    }
    hist[tid] = 0;
    hist[tid + THREADS] = 0;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
        lo = min(lo, wred[w][0]);
        hi = max(hi, wred[w][1]);
    }
    thr = lo;
    take_ties = k;
    int top = lo == hi ? 0 : 32 - __clz((int)(lo ^ hi));  // bits still open; the higher ones are settled
    int kr = k;
    uint32_t prefix = top >= 32 ? 0u : hi >> top << top;
    while (top > 0) {  // each pass settles at least one bit
        const int shift = max(top - BITS, 0);
        const uint32_t settled = top >= 32 ? 0u : ~0u << top;
#pragma unroll
        for (int i = 0; i < GPW; ++i)
            if (key[i] != kNotCand && (key[i] & settled) == prefix)
                atomicAdd(&hist[(key[i] >> shift) & (BINS - 1) & ~(settled >> shift)], 1);
        __syncthreads();
        // the bin where the count of larger keys reaches kr: thread t holds the bins 2t and 2t + 1 from the top
        const int c0 = hist[BINS - 1 - 2 * tid], c1 = hist[BINS - 2 - 2 * tid];
        int incl = c0 + c1;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int y = __shfl_up(incl, o, 64);
            if (lane >= o) incl += y;
        }
        if (lane == 63) wred[wave][0] = (uint32_t)incl;
        __syncthreads();
        int before = 0;  // keys in the bins of the waves before
#pragma unroll
        for (int w = 0; w < WAVES; ++w) before += w < wave ? (int)wred[w][0] : 0;
        const int above = before + incl - c0 - c1;
        if (above < kr && above + c0 + c1 >= kr) {
            const bool first = above + c0 >= kr;
            sel[0] = (uint32_t)(first ? BINS - 1 - 2 * tid : BINS - 2 - 2 * tid);
            sel[1] = (uint32_t)(kr - (first ? above : above + c0));
            sel[2] = (uint32_t)(first ? c0 : c1);
            sel[3] = 0u;
        }
        hist[BINS - 1 - 2 * tid] = 0;
        hist[BINS - 2 - 2 * tid] = 0;
        __syncthreads();
        prefix |= sel[0] << shift;
        kr = (int)sel[1];
        const int cnt = (int)sel[2];
        top = shift;
        thr = prefix;
        take_ties = kr;
        if (top == 0) break;
        if (cnt <= 64) {  // few keys left: rank them all against all
            const uint32_t sd = ~0u << top;
#pragma unroll
            for (int i = 0; i < GPW; ++i)
                if (key[i] != kNotCand && (key[i] & sd) == prefix) list[atomicAdd(&sel[3], 1u)] = key[i];
            __syncthreads();
            if (wave == 0) {
                const uint32_t mine = lane < cnt ? list[lane] : 0u;
                int gt = 0, ge = 0;  // larger, and larger or equal
                for (int j = 0; j < cnt; ++j) {
                    const uint32_t o = list[j];
                    gt += o > mine;
                    ge += o >= mine;
                }
                if (lane < cnt && gt < kr && ge >= kr) {  // every lane holding the k-th key writes the same
                    sel[0] = mine;
                    sel[1] = (uint32_t)(kr - gt);
                }
            }
            __syncthreads();
            thr = sel[0];
            take_ties = (int)sel[1];
            break;
        }
        __syncthreads();  // sel is rewritten by the next pass
    }
}

template <int WAVES, int GPW>
__global__ __launch_bounds__(64 * WAVES) void select_kernel(Shape s, const float* __restrict__ s_vis,
                                                          const float* __restrict__ s_txt,
                                                          const int32_t* __restrict__ budgets,
                                                          const int64_t* __restrict__ idx_off,
                                                          int32_t* __restrict__ idx) {
    __shared__ int hist[2 * 64 * WAVES];
    __shared__ uint32_t list[64];
    __shared__ uint32_t wred[WAVES][2];
    __shared__ uint32_t sel[4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int gi = blockIdx.x % s.ngroups;
    const int bl = blockIdx.x / s.ngroups;
    const int bgt = budgets[bl];
    int32_t* out = idx + idx_off[bl] + (int64_t)gi * bgt;
    // each wave's contiguous run of 64-position groups
    const int ngrp = (s.N + 63) >> 6;
    const int gpw = (ngrp + WAVES - 1) / WAVES;  // <= GPW
    const int g0 = wave * gpw, g1 = min(g0 + gpw, ngrp);

    // every score of the row is fetched at once, whatever the mode will make of it (the text scores
    // only at text positions, the vision scores only at vision positions; clamped, so each load is issued)
    const float* sv = s_vis + ((size_t)bl * s.ngroups + gi) * s.Nv;
    const float* st = s_txt + ((size_t)bl * s.ngroups + gi) * s.Nt;
    float sc[GPW];
#pragma unroll
    for (int i = 0; i < GPW; ++i) {
        const int p = min((g0 + i) * 64 + lane, s.N - 1);
        const bool vis = p >= s.Ns && p < s.Ns + s.Nv;
        sc[i] = *(vis ? sv + (p - s.Ns) : st + (p < s.Ns ? p : p - s.Nv));
    }
    int k, nc;
    const RowCtx c = row_ctx(s, s_vis, s_txt, bl, gi, bgt, k, nc);
    uint32_t key[GPW];
    uint32_t outright = 0u;  // bit i: position i of the lane is kept without competing
#pragma unroll
    for (int i = 0; i < GPW; ++i) {
        const int p = (g0 + i) * 64 + lane;
        key[i] = kNotCand;
        if (g0 + i < g1 && p < s.N) {
            if (c.kept_outright(p)) outright |= 1u << i;
            else if (c.cand(p)) key[i] = c.key_of(p, sc[i]);
        }
    }

    uint32_t thr;
    int take_ties;
    if (k <= 0) { thr = 0xFFFFFFFFu; take_ties = 0; }
    else if (k >= nc) { thr = 0u; take_ties = nc; }
    else select_threshold<WAVES, GPW>(key, k, hist, list, wred, sel, thr, take_ties);

    // ordered emission (see the header): count, one barrier, rank and write
    const unsigned long long below = (1ull << lane) - 1ull;
    int nt = 0, nk = 0;  // the wave's ties and other kept positions
#pragma unroll
    for (int i = 0; i < GPW; ++i) {
        const bool other = (outright >> i & 1u) || (key[i] != kNotCand && key[i] > thr);
        nt += __popcll(__ballot(key[i] != kNotCand && key[i] == thr));
        nk += __popcll(__ballot(other));
    }
    __syncthreads();  // wred was read by every wave
    if (lane == 0) {
        wred[wave][0] = (uint32_t)nt;
        wred[wave][1] = (uint32_t)nk;
    }
    __syncthreads();
    int tb = 0, ob = 0;  // ties and other kept positions before this wave's run
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
        tb += w < wave ? (int)wred[w][0] : 0;
        ob += w < wave ? (int)wred[w][1] : 0;
    }
#pragma unroll
    for (int i = 0; i < GPW; ++i) {
        const bool other = (outright >> i & 1u) || (key[i] != kNotCand && key[i] > thr);
        const bool tie = key[i] != kNotCand && key[i] == thr;
        const unsigned long long tm = __ballot(tie);
        const bool keep = other || (tie && tb + __popcll(tm & below) < take_ties);
        const unsigned long long km = __ballot(keep);
        const int pos = ob + min(take_ties, tb) + __popcll(km & below);
        if (keep && pos < bgt) out[pos] = (g0 + i) * 64 + lane;
        tb += __popcll(tm);
        ob += __popcll(__ballot(other));
    }
}

}  // namespace

hipError_t launch_select(const Shape& s, const float* s_vis, const float* s_txt, const int32_t* budgets,
                         const int64_t* idx_off, int32_t* idx, hipStream_t st) {
    const long long nblk = (long long)s.B * s.L * s.ngroups;
    if (nblk == 0) return hipSuccess;
    const int groups = (s.N + 63) / 64;
    const dim3 grid((unsigned)nblk);
    auto launch = [&](auto kernel, int waves) {
        hipLaunchKernelGGL(kernel, grid, dim3(64 * waves), 0, st, s, s_vis, s_txt, budgets, idx_off, idx);
    };
    // 4 waves up to 768 positions, 8 up to 3072, else 16: fewer waves meet at their barriers sooner and
    // more rows share a CU, more waves hold longer rows.  1 row of 168 positions 3.9 us (16 waves
    // 5.5); 490 rows of 558 7.1 (9.1); 128 rows of 999 6.1 by 4 waves, 5.6 by 8, 6.5 by 16; of 2979 10.7,
    // 8.3, 8.9; 224 rows of 4064 12.2 by 8, 10.5 by 16 (replayed from a graph).
    if (groups <= 4) launch(select_kernel<4, 1>, 4);
    else if (groups <= 8) launch(select_kernel<4, 2>, 4);
    else if (groups <= 12) launch(select_kernel<4, 3>, 4);
    else if (groups <= 16) launch(select_kernel<8, 2>, 8);
    else if (groups <= 24) launch(select_kernel<8, 3>, 8);
    else if (groups <= 48) launch(select_kernel<8, 6>, 8);
    else if (groups <= 64) launch(select_kernel<16, 4>, 16);
    else if (groups <= 96) launch(select_kernel<16, 6>, 16);
    else if (groups <= 144) launch(select_kernel<16, 9>, 16);
    else if (groups <= 16 * kRegGroups) launch(select_kernel<16, kRegGroups>, 16);
    else launch(select_long_kernel, kWaves);
    return hipGetLastError();
}

}  // namespace tgvkv
