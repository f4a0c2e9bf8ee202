// Gate scoring and causal top-k (paper Section 2; Appendix C.1, fused top-k selection: scores are
// produced tile by tile and never written to memory).
//
// Scores are fp32-accurate: the fp32 centroids are split into bf16 terms hi + mid + lo (24 mantissa
// bits); the queries are bf16, every product is exact in fp32.  A wave owns 16 QT consecutive queries
// and works alone -- no workgroup barrier anywhere; the four waves of a workgroup only share the L1.
//
// Few candidates (at most 320 blocks, see kGateFew): the exact scores of 16 queries are computed once, into
// registers, and the threshold with exactly k scores above it is searched there.
//
// Many candidates, two sweeps instead of keeping the scores:
//  1. hi term only: a lane keeps the maxima of GR groups of its blocks.  A query has 4 GR groups; at
//     least k of its scores reach the k-th largest of their maxima (each group's maximum is a score of
//     its own), and not many more do while 4 GR is well above k and the best blocks lie in different groups.
//     Neighbouring blocks are often alike, so 32 (rows up to 8) or 128 blocks in a row lie in different groups: one
//     maximum per score where groups of four neighbours take half of one, 2 % of the kernel, but on centroids
//     smoothed over 32 blocks those overflow (4096 blocks of 32, d = 64, k = 8, 4 heads: 1697 us, now 894; over
//     6 blocks 878 -> 785).  So that value, less the error of the
//     hi term, is a lower bound of the k-th largest score (kSumError: what is assumed of the matrix unit's sums).
//  2. hi + mid: every block above that bound becomes a candidate (18-bit score above the bound, block)
//     in LDS, about 1.1 to 1.5 k of them.  The k-th largest candidate is searched in registers; where
//     the next one is closer than the error of hi + mid (2^-16 of |q| |c| at d = 64, 2^-15 at 128), the candidates
//     inside that error are scored again from all three terms and ranked exactly, ties to the lower block.
// Strips that do not fit (more candidates or closer scores than there is room for: many equal scores;
// non-finite values) are put on a list for the search of topk_mfma.hip.
//
// What bounds it: VALU issue in the sweeps (per 16 x 16 scores 4 instructions in the first, about 5 in the second,
// against d / 32 and d / 16 MFMAs) and the searches.  The kernel before it, a histogram of all scores by LDS
// atomics and an exact three-term sweep, took 46 us at N = 8192, B = 128, k = 8, 16 heads (now 29), 22.3 ms
// at N = 524288, B = 128, k = 8, 32 slices (now 15.4 + 0.3) and 4.4 ms at N = 131072, d = 128, B = 64,
// k = 32, 16 heads (now 3.4 + 0.3).
#include <algorithm>
#include <type_traits>

#include "gate.h"

namespace moba {

// Classes by the longest row of kept blocks, 8 and 32 (where each runs: gate_supported()).  A wave takes 16 QT
// queries: more of them share every operand load, but their candidates (SEG per half query) cap the waves per
// compute unit, and the kernel lives on waves: at N = 524288, B = 128, k = 8 it takes 23.7 ms with two waves per
// SIMD and 15.4 with three.
template <int KC> struct GateCfg;
template <> struct GateCfg<8> {
    static constexpr int QT = 4, GR = 8, SEG = 24;
};
template <> struct GateCfg<32> {
    static constexpr int QT = 2, GR = 32, SEG = 72;
};
// tiles of 16 blocks whose scores a wave keeps in registers: as many as three waves per SIMD (d = 128: two,
// the operands are larger) leave room for
template <int D> constexpr int kGateFew = D == 64 ? 20 : 16;
constexpr int kGateWaves = 4;
constexpr int kGateBand = 64;                     // candidates of a strip that can be scored again
constexpr int kGateIdBits = 14;
constexpr int kGateTopKey = 262141;                // keys are 1 .. kGateTopKey + 1 < 2^18 - 1
constexpr float kGateKeys = (float)kGateTopKey;

template <int KC>
struct GateLds {                                  // words per wave
    using C = GateCfg<KC>;
    static constexpr int CAND = 16 * C::QT * 2 * C::SEG;
    static constexpr int BAND = kGateBand * 2;
    static constexpr int WORDS = CAND + BAND + kGateBand + 16 * C::QT;
};

// c3 <- the three bf16 terms of the fp32 centroids, in MFMA operand order: the 16 bytes lane (m, g)
// feeds to the MFMA for blocks 16 jt + m, channels 32 ks + 8 g .. + 8, term t, sit at
// (((slice * ntile + jt) * 3 + t) * (D / 32) + ks) * 1024 + 16 * lane, so that one load instruction of a
// wave covers 1 KB of consecutive bytes.  Blocks beyond n read as zero.
// norms[slice * 16 ntile + block] <- (|c - hi|, |c - hi - mid|, |c|).  A wave per tile.
template <int D>
__global__ __launch_bounds__(256) void split3_kernel(const float* __restrict__ c, bf16_t* __restrict__ out,
                                                     float4* __restrict__ norms, int32_t* __restrict__ redo, int n,
                                                     int ntile, int tiles_total)
{
    constexpr int KS = D / 32;
    if (redo && blockIdx.x == 0 && threadIdx.x == 0) redo[0] = 0;
    const int tile = blockIdx.x * 4 + threadIdx.x / kWave, lane = threadIdx.x % kWave;
    if (tile >= tiles_total) return;
    const int jt = tile % ntile, row = 16 * jt + (lane & 15), g = lane >> 4;
    const int64_t s = tile / ntile;
    float n1 = 0.f, n2 = 0.f, nc = 0.f;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
        float x[8], t[3][8];
        if (row < n) Vec8<float>::load(c + (s * n + row) * D + 32 * ks + 8 * g, x);
        else {
#pragma unroll
            for (int e = 0; e < 8; ++e) x[e] = 0.f;
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float hi = bf16_to_f32(f32_to_bf16(x[e])), r1 = x[e] - hi;
            const float mid = bf16_to_f32(f32_to_bf16(r1)), r2 = r1 - mid;
            t[0][e] = hi; t[1][e] = mid; t[2][e] = r2;
            n1 = fmaf(r1, r1, n1); n2 = fmaf(r2, r2, n2); nc = fmaf(x[e], x[e], nc);
        }
#pragma unroll
        for (int term = 0; term < 3; ++term) {
            bf16_t o[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) o[e] = f32_to_bf16(t[term][e]);
            *reinterpret_cast<uint4*>(out + (((int64_t)tile * 3 + term) * KS + ks) * 512 + lane * 8) = *reinterpret_cast<const uint4*>(o);
        }
    }
    if (norms) {
        n1 = fsum_g(n1); n2 = fsum_g(n2); nc = fsum_g(nc);
        if (g == 0) norms[s * 16 * ntile + row] = make_float4(sqrtf(n1), sqrtf(n2), sqrtf(nc), 0.f);
    }
}

// Tiles [tlo, thi) of a sweep: f(u, tile, sc) with u = (tile - tlo) mod UN, a compile-time number;
// sc[qt][i] is the score of query 16 qt + m16 against block 16 tile + 4 g + i from terms 0 .. TOP,
// smallest first.  The operands of W tiles are loaded while the W tiles before them are worked on (an L2
// round trip is several tiles long).  The scheduling barriers and the empty asm statement keep the
// compiler from moving the loads down to their first use.
template <int D, int TOP, int QT, int UN, int W, typename F>
__device__ __forceinline__ void gate_sweep(const char* __restrict__ c3s, int tlo, int thi, const Frag (&qb)[QT][D / 32],
                                           int lane, F f)
{
    constexpr int KS = D / 32;
    static_assert(UN % (2 * W) == 0, "two operand sets");
    if (tlo >= thi) return;
    Frag a[2][W][TOP + 1][KS];
    const uint32_t mine = (uint32_t)lane * 16u;              // (scalar base + 32-bit lane offset: no address arithmetic per load)
    auto load = [&](int buf, int t) {
#pragma unroll
        for (int v = 0; v < W; ++v) {
            const char* tb = c3s + (int64_t)min(t + v, thi - 1) * (3 * KS * 1024);
#pragma unroll
            for (int term = 0; term <= TOP; ++term)
#pragma unroll
                for (int ks = 0; ks < KS; ++ks)
                    a[buf][v][term][ks].q = *reinterpret_cast<const uint4*>(tb + (term * KS + ks) * 1024 + mine);
        }
    };
    load(0, tlo);
    for (int t = tlo; t < thi; t += UN) {
#pragma unroll
        for (int u = 0; u < UN; u += W)
            if (t + u < thi) {
                const int buf = u / W % 2;
                load(buf ^ 1, t + u + W);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int v = 0; v < W; ++v)
                    if (v == 0 || t + u + v < thi) {
                        f32x4_t sc[QT];
#pragma unroll
                        for (int qt = 0; qt < QT; ++qt) sc[qt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                        for (int term = TOP; term >= 0; --term)
#pragma unroll
                            for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                                for (int qt = 0; qt < QT; ++qt) sc[qt] = mfma16(a[buf][v][term][ks], qb[qt][ks], sc[qt]);
                        f(u + v, t + u + v, sc);
                    }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int v = 0; v < W; ++v)
#pragma unroll
                    for (int term = 0; term <= TOP; ++term)
#pragma unroll
                        for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+v"(a[buf ^ 1][v][term][ks].n));
            }
    }
}

// Strips of 16 queries with at most 16 TA candidate blocks, wave `at` of a slice
template <int D, int TA>
__device__ __forceinline__ void few_strip(const bf16_t* __restrict__ Q, const bf16_t* __restrict__ c3, int ntile_all,
                                          int32_t* __restrict__ idx, int N, int B, int k, int strips, int s, int at, int G,
                                          const int32_t* __restrict__ blk_first, uint32_t* lds)
{
    constexpr int KS = D / 32;
    const int lane = threadIdx.x % kWave;
    const int m16 = lane & 15, g = lane >> 4;
    const int strip = strips - 1 - at;           // late strips, with the most candidates, first
    if (strip < 0) return;
    const int t0 = 16 * strip, rows_here = min(16, N - t0);
    const int pfirst = t0 / B, pmax = (t0 + rows_here - 1) / B;
    const int fmin = blk_first ? blk_first[pfirst] : 0, fmax = blk_first ? blk_first[pmax] : 0;
    const int tbeg = fmin / 16, tend = (pmax + 15) / 16;
    if (tend - tbeg > TA) return;
    const int ilo = (fmax + 15) / 16, ihi = pfirst / 16;                // tiles that are candidates of every query
    Frag q[1][KS];
    const int64_t qrow = (int64_t)s * N + min(t0 + m16, N - 1);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) q[0][ks].q = *reinterpret_cast<const uint4*>(Q + qrow * D + 8 * g + 32 * ks);
    const int own = m16 < rows_here ? (t0 + m16) / B : 0;
    const int first = blk_first && m16 < rows_here ? blk_first[own] : 0;
    const char* c3s = reinterpret_cast<const char*>(c3) + (int64_t)(s / G) * ntile_all * (3 * KS * 1024);
    f32x4_t x[TA];
#pragma unroll
    for (int u = 0; u < TA; ++u) x[u] = f32x4_t{-INFINITY, -INFINITY, -INFINITY, -INFINITY};
    ScoreStats st;
    gate_sweep<D, 2, 1, TA, 1>(c3s, tbeg, tend, q, lane, [&](int u, int jt, const f32x4_t (&sc)[1]) {
        st.fold(sc[0], x[u], jt < ilo || jt >= ihi, 16 * jt + 4 * g - first, own - first);
    });
    st.tame<TA>(x, tend - tbeg, 16 * tbeg + 4 * g - first, own - first);
    select_and_stage<TA>(x, st, tend - tbeg, tbeg, min(k, own - first), own - first, k, lds, lane);
    store_rows(reinterpret_cast<const int32_t*>(lds), idx + ((int64_t)s * N + t0) * k, rows_here, k, lane);
}

// every strip of the call has few candidates
template <int D, int TA>
__global__ __launch_bounds__(kGateWaves * kWave) __attribute__((amdgpu_waves_per_eu(D == 64 ? 3 : 2)))
void gate_few_kernel(
    const bf16_t* __restrict__ Q, const bf16_t* __restrict__ c3, int ntile_all, int32_t* __restrict__ idx, int N, int B,
    int k, int strips, int bh, int G, const int32_t* __restrict__ blk_first)
{
    extern __shared__ __align__(16) uint32_t gate_lds[];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    int s, pos;
    if (!schedule(blockIdx.x, bh, (strips + kGateWaves - 1) / kGateWaves, s, pos)) return;
    few_strip<D, TA>(Q, c3, ntile_all, idx, N, B, k, strips, s, pos * kGateWaves + wave, G, blk_first,
                     gate_lds + wave * select_words<TA>(k));
}

// Rows of many candidates and, in the last workgroups of every slice, those of few: in one launch the few ones fill
// what the last of the many leave idle.
template <int D, int KC>
__global__ __launch_bounds__(kGateWaves * kWave) __attribute__((amdgpu_waves_per_eu(D == 64 ? 3 : 2)))
void gate_many_kernel(
    const bf16_t* __restrict__ Q, const bf16_t* __restrict__ c3,
    const float4* __restrict__ norms, int ntile_all, int32_t* __restrict__ idx, int32_t* __restrict__ redo, int N, int B,
    int n, int k, int strips, int many_wgs, int few_strips, int few_wgs, int bh, int G, const int32_t* __restrict__ blk_first)
{
    using C = GateCfg<KC>;
    using L = GateLds<KC>;
    constexpr int KS = D / 32, QT = C::QT, SEG = C::SEG;
    extern __shared__ __align__(16) uint32_t gate_lds[];
    const int lane = threadIdx.x % kWave, wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int m16 = lane & 15, g = lane >> 4;
    uint32_t* cand = gate_lds + wave * L::WORDS;
    uint2* band = reinterpret_cast<uint2*>(cand + L::CAND);             // (exact key, query << 16 | block)
    uint32_t* band_keep = reinterpret_cast<uint32_t*>(band + kGateBand);
    int* band_want = reinterpret_cast<int*>(band_keep + kGateBand);     // [16 QT] band candidates a query still wants

    int s, pos;
    if (!schedule(blockIdx.x, bh, many_wgs + few_wgs, s, pos)) return;
    if (pos >= many_wgs) {
        static_assert(L::WORDS >= select_words<kGateFew<D>>(KC), "one LDS region per wave for both");
        few_strip<D, kGateFew<D>>(Q, c3, ntile_all, idx, N, B, k, few_strips, s, (pos - many_wgs) * kGateWaves + wave, G,
                               blk_first, cand);
        return;
    }
    const int strip = strips - 1 - (pos * kGateWaves + wave);           // late strips, with the most candidates, first
    if (strip < 0) return;
    const int t0 = strip * 16 * QT, rows_here = min(16 * QT, N - t0);
    const char* c3s = reinterpret_cast<const char*>(c3) + (int64_t)(s / G) * ntile_all * (3 * KS * 1024);
    int32_t* out = idx + ((int64_t)s * N + t0) * k;

    const int pfirst = t0 / B, pmax = (t0 + rows_here - 1) / B;
    // (the queries of a strip are consecutive: first and own block of the first query are the smallest)
    const int fmin = blk_first ? blk_first[pfirst] : 0, fmax = blk_first ? blk_first[pmax] : 0;
    const int tbeg = fmin / 16, tend = (pmax + 15) / 16;
    const int ilo = (fmax + 15) / 16, ihi = pfirst / 16;                // tiles that are candidates of every query
    auto load_q = [&](int qt, Frag (&q)[KS]) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const int64_t r = min(t0 + 16 * qt + m16, N - 1);
            q[ks].q = *reinterpret_cast<const uint4*>(Q + ((int64_t)s * N + r) * D + 8 * g + 32 * ks);
        }
    };
    int32_t* stage = reinterpret_cast<int32_t*>(cand);                  // [16][k + 1] rows on their way out

    if (tend - tbeg <= kGateFew<D>) return;                                // (few_strip's)

    int own[QT], first[QT], need[QT];                                   // candidates of a query: blocks first .. own - 1
#pragma unroll
    for (int qt = 0; qt < QT; ++qt) {
        const int q = 16 * qt + m16;
        own[qt] = q < rows_here ? (t0 + q) / B : 0;
        first[qt] = blk_first && q < rows_here ? blk_first[own[qt]] : 0;
        need[qt] = min(k, own[qt] - first[qt]);
    }
    Frag qb[QT][KS];
#pragma unroll
    for (int qt = 0; qt < QT; ++qt) load_q(qt, qb[qt]);

    // hands the 64 queries around this strip to the search (which numbers them from the last on)
    auto search_again = [&]() {
        const int per_slice = (N + 63) / 64;
        if (lane == 0) redo[1 + atomicAdd(redo, 1)] = s * per_slice + per_slice - 1 - t0 / 64;
    };

    // ---- many candidates.  Errors of the approximate scores against the three-term ones: |q . (c - hi)|
    // <= |q| |c - hi|, plus what the fp32 sums of both can lose.  Every product is exact, and in whatever order the
    // matrix unit adds them, an addition is taken to lose at most 2^-23 of the largest number in it (cutting off
    // what does not fit; rounding to nearest would halve that).  The terms go smallest first, so only the D
    // additions of the hi term meet numbers of the size of |q| |c|; those of the others lose 2^-8 and 2^-16 as
    // much: less than 1.02 D 2^-23 |q| |c| per score, twice that for the difference of two.
    constexpr float kSumError = 2.04f * D / 8388608.f;
    float qn[QT], e1, e2;                                               // |q|; errors per |q| of one and of two terms
    {
        float r1 = 0.f, r2 = 0.f, rc = 0.f;
        const float4* nr = norms + (int64_t)(s / G) * 16 * ntile_all;
        for (int j = 16 * tbeg + lane; j < 16 * tend; j += kWave) {
            const float4 v = nr[j];
            r1 = max_nan(r1, v.x); r2 = max_nan(r2, v.y); rc = max_nan(rc, v.z);
        }
#pragma unroll
        for (int o = 1; o < kWave; o <<= 1) {
            r1 = max_nan(r1, __shfl_xor(r1, o, kWave));
            r2 = max_nan(r2, __shfl_xor(r2, o, kWave));
            rc = max_nan(rc, __shfl_xor(rc, o, kWave));
        }
        const float acc = kSumError * rc;
        auto uniform = [](float x) { return __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(x))); };
        e1 = uniform(1.001f * r1 + acc);
        e2 = uniform(1.001f * r2 + acc);
        bool finite = true;
#pragma unroll
        for (int qt = 0; qt < QT; ++qt) {
            float q2 = 0.f;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float a = __uint_as_float(qb[qt][ks].u[e] << 16), b = __uint_as_float(qb[qt][ks].u[e] & 0xffff0000u);
                    q2 = fmaf(a, a, fmaf(b, b, q2));
                }
            qn[qt] = sqrtf(fsum_g(q2));
            finite = finite && qn[qt] * e1 < 1e37f && qn[qt] * rc < 1e37f;
        }
        if (__ballot(!finite)) {
            search_again();
            return;
        }
    }
    // (a floor under both: kGateKeys / error stays finite for a query of zeros as well)
    auto error = [&](float per, int qt) { return fmaf(qn[qt], per, 1e-30f); };
    auto mask_edges = [&](int jt, f32x4_t (&sc)[QT]) {                  // blocks that are no candidates: -inf
        if (jt >= ilo && jt < ihi) return;
#pragma unroll
        for (int qt = 0; qt < QT; ++qt) {
            const int j0 = 16 * jt + 4 * g - first[qt];
#pragma unroll
            for (int i = 0; i < 4; ++i)
                sc[qt][i] = (uint32_t)(j0 + i) < (uint32_t)(own[qt] - first[qt]) ? sc[qt][i] : -INFINITY;
        }
    };
    // sweep 1: group maxima
    float scale[QT], base[QT], thr[QT];                                 // key of a score: (score - base) * scale + 1.5; collected from thr on
    {
        f32x4_t gm[QT][C::GR / 4];
#pragma unroll
        for (int qt = 0; qt < QT; ++qt)
#pragma unroll
            for (int u = 0; u < C::GR / 4; ++u) gm[qt][u] = f32x4_t{-INFINITY, -INFINITY, -INFINITY, -INFINITY};
        gate_sweep<D, 0, QT, C::GR, 2>(c3s, tbeg, tend, qb, lane, [&](int u, int jt, f32x4_t (&sc)[QT]) {
            mask_edges(jt, sc);
#pragma unroll
            for (int qt = 0; qt < QT; ++qt)
#pragma unroll
                for (int i = 0; i < 4; ++i) gm[qt][u % (C::GR / 4)][i] = max_nan(sc[qt][i], gm[qt][u % (C::GR / 4)][i]);
        });
#pragma unroll
        for (int qt = 0; qt < QT; ++qt) {
            float mx = -INFINITY, mn = INFINITY, sum = 0.f, sq = 0.f;
            int some = 0;
#pragma unroll
            for (int u = 0; u < C::GR / 4; ++u)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float v = gm[qt][u][i];
                    mx = fmaxf(mx, v);
                    mn = fminf(mn, v == -INFINITY ? INFINITY : v);
                    const bool in = v > -INFINITY;
                    some += (int)in;
                    sum += in ? v : 0.f;
                    sq = in ? fmaf(v, v, sq) : sq;
                }
            mx = fmax_g(mx);
            float lo = fmin_g(mn), hi = mx + fabsf(mx) * 1e-6f + 1e-30f;
            Bracket b = {sum_g(some), 0};
            // (fewer groups with candidates than blocks to keep: all of its candidates are collected)
            const bool all = b.clo < need[qt] || need[qt] == own[qt] - first[qt];
            if (all) b.clo = need[qt];
            const float inv = 1.f / (float)max(b.clo, 1), mean = fsum_g(sum) * inv;
            const float var = fmaxf(fsum_g(sq) * inv - mean * mean, 0.f);
            search_threshold<C::GR / 4>(gm[qt], C::GR / 4, need[qt], need[qt] >> 4, 0,
                                        mean + sqrtf(var) * normal_quantile(((float)need[qt] + 0.5f) * inv), lo, hi, b);
            const float e = error(e1, qt) + error(e2, qt);
            // (Keys of an `all` query tell nothing
            // apart beyond their block: it keeps every candidate or goes to the exact ranking.)
            scale[qt] = all ? 0.f : kGateKeys / (mx - lo + 3.f * e);
            thr[qt] = all ? (16 * qt + m16 < rows_here ? -kFltMax : kFltMax) : lo - e;   // (rows past the last: nothing)
            base[qt] = all ? 0.f : thr[qt];                              // (the difference first: no key falls below 1)
        }
    }
    // sweep 2: candidates.  The lanes g = 2 p and 2 p + 1 of a query fill the segment p of SEG words from
    // its two ends.
    const int dir = (g & 1) ? -1 : 1;
    uint32_t at[QT], at0[QT];                                           // next place, first place
    float from[QT];                                                     // collect from here on; INFINITY: no room for a tile's four
    bool full = false;
#pragma unroll
    for (int qt = 0; qt < QT; ++qt) {
        const uint32_t seg = (uint32_t)(((16 * qt + m16) * 2 + (g >> 1)) * SEG);
        at0[qt] = at[qt] = (g & 1) ? seg + SEG - 1 : seg;
        from[qt] = thr[qt];
    }
    gate_sweep<D, 1, QT, 2, 1>(c3s, tbeg, tend, qb, lane, [&](int, int jt, f32x4_t (&sc)[QT]) {
        mask_edges(jt, sc);
        const uint32_t id = 16 * jt + 4 * g;
        // (all compares first: a scalar branch right behind its compare waits for it every time)
        uint64_t hits[QT][4];
#pragma unroll
        for (int qt = 0; qt < QT; ++qt)
#pragma unroll
            for (int i = 0; i < 4; ++i) hits[qt][i] = __ballot(sc[qt][i] >= from[qt]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int qt = 0; qt < QT; ++qt) {
            const uint64_t any = hits[qt][0] | hits[qt][1] | hits[qt][2] | hits[qt][3];
            if (any == 0) continue;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (KC == 8 && hits[qt][i] == 0) continue;             // (few of many: most scores end here)
                if (__builtin_amdgcn_inverse_ballot_w64(hits[qt][i])) {
                    const uint32_t key = min((uint32_t)fmaf(sc[qt][i] - base[qt], scale[qt], 1.5f), (uint32_t)kGateTopKey + 1u);
                    cand[at[qt]] = (key << kGateIdBits) + (id + i);
                    at[qt] += dir;
                }
            }
            const uint32_t n_here = (g & 1) ? at0[qt] - at[qt] : at[qt] - at0[qt];
            if (n_here > (uint32_t)(SEG - 4)) from[qt] = INFINITY;
        }
    });
    int cnt[QT];
#pragma unroll
    for (int qt = 0; qt < QT; ++qt) cnt[qt] = (int)((g & 1) ? at0[qt] - at[qt] : at[qt] - at0[qt]);
    __builtin_amdgcn_wave_barrier();
    // the candidates of a query come into the registers of its lanes, alternate ones to the two lanes of a pair
    uint32_t y[QT][SEG / 2];
    int total[QT];
#pragma unroll
    for (int qt = 0; qt < QT; ++qt) {
        const int other = __shfl_xor(cnt[qt], 16, kWave), pair = cnt[qt] + other;
        const int up = (g & 1) ? other : cnt[qt];                       // entries from the front
        full = full || from[qt] == INFINITY || pair > SEG;
        const uint32_t* seg = cand + ((16 * qt + m16) * 2 + (g >> 1)) * SEG;
#pragma unroll
        for (int j = 0; j < SEG / 2; ++j) {
            const int p = 2 * j + (g & 1);
            const uint32_t v = seg[p < up ? p : min(max(SEG - pair + p, 0), SEG - 1)];
            y[qt][j] = p < pair ? v : 0u;
        }
        total[qt] = sum_g(cnt[qt]);
        full = full || total[qt] < need[qt];                            // (cannot be, see kSumError)
    }
    // The k-th largest candidate; where the next one is within `width` of it, those within `width` of the k-th go on
    // the band: scored again from all three terms, in the order of the other kernels, so that all agree on close ones.
    // Those above stay in, those below out, the band decides the rest.
    uint32_t cut[QT];
    int nband = 0, upto[QT];                                            // the same in all lanes
    if (!__ballot(full)) {
#pragma unroll
        for (int qt = 0; qt < QT; ++qt) {
            cut[qt] = search_key<SEG / 2>(y[qt], 1u << kGateIdBits, 0xffffffffu, need[qt], total[qt]);
            upto[qt] = nband;
            uint32_t kth = 0xffffffffu, next = 0u;
#pragma unroll
            for (int j = 0; j < SEG / 2; ++j) {
                kth = min(kth, y[qt][j] >= cut[qt] ? y[qt][j] : 0xffffffffu);
                next = max(next, y[qt][j] < cut[qt] ? y[qt][j] : 0u);
            }
            kth = umin_g(kth) >> kGateIdBits;
            next = umax_g(next) >> kGateIdBits;
            const uint32_t width = (uint32_t)fminf(2.f * error(e2, qt) * scale[qt], kGateKeys) + 2u;
            const bool close = need[qt] > 0 && total[qt] > need[qt] && kth - next <= width;
            if (!__ballot(close)) continue;
            const uint32_t blo = !close ? 1u : kth > width ? kth - width : 1u;      // (not close: no key lies between)
            const uint32_t bhi = !close ? 0u : min(kth + width, (uint32_t)kGateTopKey + 1u);
            int sure = 0;
#pragma unroll
            for (int j = 0; j < SEG / 2; ++j) {
                const uint32_t key = y[qt][j] >> kGateIdBits;
                sure += (int)(key > bhi);
                const bool in = key >= blo && key <= bhi;
                const uint64_t m = __ballot(in);
                if (m == 0) continue;
                const int p = nband + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
                if (in && p < kGateBand) band[p].y = (uint32_t)(16 * qt + m16) << 16 | (y[qt][j] & ((1u << kGateIdBits) - 1u));
                nband += __popcll(m);
            }
            upto[qt] = nband;
            sure = sum_g(sure);
            if (close) {
                cut[qt] = (bhi + 1u) << kGateIdBits;
                if (g == 0) band_want[16 * qt + m16] = need[qt] - sure;
            }
        }
    }
    if (__ballot(full) || nband > kGateBand) {
        search_again();
        return;
    }
    __builtin_amdgcn_wave_barrier();
    if (nband > 0) {
        int at_band = 0;
#pragma unroll
        for (int qt = 0; qt < QT; ++qt)
#pragma unroll 1
            for (; at_band < upto[qt]; ++at_band) {
                const uint32_t what = (uint32_t)__builtin_amdgcn_readfirstlane((int)band[at_band].y);
                const int blk = (int)(what & 0xffffu), in = blk & 15;
                const char* tb = c3s + (int64_t)(blk >> 4) * (3 * KS * 1024) + lane * 16;
                f32x4_t sc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int term = 2; term >= 0; --term)
#pragma unroll
                    for (int ks = 0; ks < KS; ++ks) {
                        Frag a;
                        a.q = *reinterpret_cast<const uint4*>(tb + (term * KS + ks) * 1024);
                        sc = mfma16(a, qb[qt][ks], sc);
                    }
                const float mine = in & 2 ? (in & 1 ? sc[3] : sc[2]) : (in & 1 ? sc[1] : sc[0]);
                if (lane == 4 * (in & 12) + (int)((what >> 16) & 15u)) band[at_band].x = order_key(mine);
            }
    }
    __builtin_amdgcn_wave_barrier();
    if (nband > 0) {
        // a lane per band candidate ranks it among those of its query
        const uint2 me = lane < nband ? band[lane] : make_uint2(0u, 0u);
        int rank = 0;
        for (int o = 0; o < nband; ++o) {
            const uint2 x = band[o];
            rank += (int)((x.y >> 16) == (me.y >> 16) && (x.x > me.x || (x.x == me.x && x.y < me.y)));
        }
        if (lane < nband) band_keep[lane] = rank < band_want[me.y >> 16] ? me.y : 0xffffffffu;
        __builtin_amdgcn_wave_barrier();
    }
    // ---- kept blocks as bit rows over the candidates' LDS, `batch` queries at a time, then ascending rows
    const int Wn = ((n + 31) / 32) | 1;                                 // words per row (odd: rows on different banks)
    uint32_t* bits = cand + 16 * (k + 1);
    const int batch = min(16, (L::CAND - 16 * (k + 1)) / Wn);
#pragma unroll
    for (int qt = 0; qt < QT; ++qt) {
        if (16 * qt >= rows_here) break;
        for (int b0 = 0; b0 < 16; b0 += batch) {
            const bool here = m16 >= b0 && m16 < b0 + batch;
            for (int i = lane; i < batch * Wn; i += kWave) bits[i] = 0u;
            __builtin_amdgcn_wave_barrier();
            uint32_t* row = bits + (m16 - b0) * Wn;
            if (here) {
#pragma unroll
                for (int j = 0; j < SEG / 2; ++j)
                    if (y[qt][j] >= cut[qt]) {
                        const uint32_t blk = y[qt][j] & ((1u << kGateIdBits) - 1u);
                        atomicOr(&row[blk >> 5], 1u << (blk & 31));
                    }
            }
            if (lane < nband) {
                const uint32_t v = band_keep[lane];
                const int q = (int)(v >> 16) - 16 * qt;
                if (v != 0xffffffffu && q >= b0 && q < min(16, b0 + batch))
                    atomicOr(&bits[(q - b0) * Wn + ((v & 0xffffu) >> 5)], 1u << (v & 31));
            }
            __builtin_amdgcn_wave_barrier();
            rows_from_bits(row, Wn, here, 0, k, stage + m16 * (k + 1), lane);
            __builtin_amdgcn_wave_barrier();
        }
        store_rows(stage, out + (int64_t)16 * qt * k, min(16, rows_here - 16 * qt), k, lane);
        __builtin_amdgcn_wave_barrier();
    }
}

// fp32 queries, at most 512 blocks: exact scores of 16 queries from v_mfma_f32_16x16x4_f32 in registers.
// The instruction is a chain of four fused multiply-adds in ascending channel, so with the channels in order
// a score is bit for bit what one lane's loop over them gives (topk_reference.hip).  A 16-byte read holds
// four channels of one lane; transpose_g spreads them over the four instructions that want them.
// Bound by the latency of few waves at these sizes: 76 us -> 15 at N = 4096, B = 64, 4 heads against the
// wave per query of topk_reference.hip.
constexpr int kGateF32Tiles = 32;

__device__ __forceinline__ f32x4_t transpose_g(f32x4_t v)               // [i] of lane group g <-> [g] of lane group i
{
    uint32_t x[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) x[i] = __float_as_uint(v[i]);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const auto h = __builtin_amdgcn_permlane32_swap(x[i], x[i + 2], false, false);
        x[i] = h[0]; x[i + 2] = h[1];
    }
#pragma unroll
    for (int i = 0; i < 4; i += 2) {
        const auto h = __builtin_amdgcn_permlane16_swap(x[i], x[i + 1], false, false);
        x[i] = h[0]; x[i + 1] = h[1];
    }
    return f32x4_t{__uint_as_float(x[0]), __uint_as_float(x[1]), __uint_as_float(x[2]), __uint_as_float(x[3])};
}

template <int D>
__global__ __launch_bounds__(kGateWaves * kWave) void gate_f32_kernel(
    const float* __restrict__ Q, const float* __restrict__ cent, int32_t* __restrict__ idx, int N, int B, int n, int k,
    int strips, int bh, int G, const int32_t* __restrict__ blk_first)
{
    constexpr int CT = D / 16;
    extern __shared__ __align__(16) uint32_t gate_lds[];
    const int lane = threadIdx.x % kWave, wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int m16 = lane & 15, g = lane >> 4;
    uint32_t* lds = gate_lds + wave * select_words<kGateF32Tiles>(k);
    int s, pos;
    if (!schedule(blockIdx.x, bh, (strips + kGateWaves - 1) / kGateWaves, s, pos)) return;
    const int strip = strips - 1 - (pos * kGateWaves + wave);
    if (strip < 0) return;
    const int t0 = 16 * strip, rows_here = min(16, N - t0);
    const int own = m16 < rows_here ? (t0 + m16) / B : 0;
    const int first = blk_first && m16 < rows_here ? blk_first[own] : 0;
    const int tbeg = (blk_first ? blk_first[t0 / B] : 0) / 16, tend = ((t0 + rows_here - 1) / B + 15) / 16;
    f32x4_t q[CT];
    const float* qr = Q + ((int64_t)s * N + min(t0 + m16, N - 1)) * D + 4 * g;
#pragma unroll
    for (int t = 0; t < CT; ++t) q[t] = transpose_g(*reinterpret_cast<const f32x4_t*>(qr + 16 * t));
    f32x4_t x[kGateF32Tiles];
    ScoreStats st;
    const float* cs = cent + (int64_t)(s / G) * n * D + 4 * g;
#pragma unroll
    for (int u = 0; u < kGateF32Tiles; ++u) {
        x[u] = f32x4_t{-INFINITY, -INFINITY, -INFINITY, -INFINITY};
        if (u < tend - tbeg) {
        f32x4_t sc = {0.f, 0.f, 0.f, 0.f};
        const float* cr = cs + (int64_t)min(16 * (tbeg + u) + m16, n - 1) * D;
#pragma unroll
        for (int t = 0; t < CT; ++t) {
            const f32x4_t a = transpose_g(*reinterpret_cast<const f32x4_t*>(cr + 16 * t));
#pragma unroll
            for (int i = 0; i < 4; ++i) sc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i], q[t][i], sc, 0, 0, 0);
        }
        st.fold(sc, x[u], true, 16 * (tbeg + u) + 4 * g - first, own - first);
        }
    }
    st.tame<kGateF32Tiles>(x, tend - tbeg, 16 * tbeg + 4 * g - first, own - first);
    select_and_stage<kGateF32Tiles>(x, st, tend - tbeg, tbeg, min(k, own - first), own - first, k, lds, lane);
    store_rows(reinterpret_cast<const int32_t*>(lds), idx + ((int64_t)s * N + t0) * k, rows_here, k, lane);
}

// ---- host ------------------------------------------------------------------------------------------

// most blocks of a call without rows of many candidates
static int few_blocks(const Dims& s) { return 16 * (s.D == 128 ? kGateFew<128> : kGateFew<64>); }

// Where these kernels run and where the histogram search of topk_mfma.hip does, both measured over
// N <= 131072 with 4 and 16 heads (us, search -> here, 16 heads where not said otherwise):
//  - scores in registers: every call it takes (d = 64, 300 blocks of 32, k = 16: 84 -> 64); very short rows up to
//    256 blocks only (300 blocks of 128, k = 3: 179 -> 193; keeping 512 blocks, d = 64, k = 3: 335 -> 576)
//  - two sweeps, rows of at most 8: enough strips to fill the chip with one wave per 64 queries (700 blocks of 32,
//    k = 8: 185 -> 167, with 4 heads 73 -> 95) and enough blocks (2048 of 64, k = 8: 1682 -> 1262; d = 128, 300 of
//    64: 162 -> 162).  Rows of 15 and 16 overflow their candidates too often (2048 of 64: 1867 -> 2390)
//  - two sweeps, rows of 17 to 32 at d = 128: from 2048 blocks on and behind a key conv of width 3 or 4 only, which
//    blurs the centroids and leaves the histogram's windows little to cut (calls with lists, k = 17 / 32; 2048 of 64:
//    width 4 4498 -> 3959 / 4653 -> 4405, width 3 4328 -> 3928 / 4545 -> 4369, width 2 4073 -> 3902 / 4430 -> 4350, none
//    3307 -> 3831 / 3621 -> 4246; 2048 of 32: width 4 2152 -> 1977 / 2299 -> 2184, width 2 1870 -> 1954 / 2036 -> 2158;
//    1000 of 64: width 4 1411 -> 1403 / 1469 -> 1543)
// Longer rows stay with the search (N = 32768, B = 32, k = 64, d = 64: 446 against 630).
bool gate_supported(const Dims& s)
{
    if (s.k <= 0 || s.k > 64 || (s.flags & (MOBA_FLAG_REFERENCE_KERNELS | MOBA_FLAG_GATE_EXACT_SEARCH))) return false;
    if (s.dtype != MOBA_BF16) return s.n <= 16 * kGateF32Tiles;
    if (s.n <= few_blocks(s)) return s.k >= 8 || s.n <= 256;
    if (s.n > (1 << kGateIdBits) || s.n < (s.D == 64 ? 513 : 448) || (int64_t)s.bh * s.N < 300000) return false;
    return s.k <= 8 || (s.D == 128 && s.k > 16 && s.k <= 32 && s.n >= 2048 && s.W >= 3);
}

// workspace: [the three terms][norms of every block][list of strips to search again: count, strips]
static bool gate_may_redo(const Dims& s) { return s.n > few_blocks(s); }
static size_t terms_bytes(const Dims& s) { return a256(3 * sizeof(bf16_t) * (size_t)s.bhk * ((s.n + 15) / 16 * 16) * s.D); }
static size_t norms_bytes(const Dims& s) { return a256(sizeof(float4) * (size_t)s.bhk * ((s.n + 15) / 16 * 16)); }
size_t gate_ws_bytes(const Dims& s)
{
    if (s.dtype != MOBA_BF16) return 256;
    // (at most two entries per 64 queries: one for each half)
    return terms_bytes(s) + (gate_may_redo(s) ? norms_bytes(s) + a256(4 * (1 + 2 * (size_t)s.bh * ((s.N + 63) / 64))) : 0);
}

hipError_t launch_split3(const Dims& s, const float* cent, bf16_t* c3, float4* norms, int32_t* redo, hipStream_t st)
{
    const int ntile = (s.n + 15) / 16, tiles = s.bhk * ntile;            // centroids: per key/value head
    const dim3 grid((unsigned)((tiles + 3) / 4));
    if (s.D == 64) hipLaunchKernelGGL(split3_kernel<64>, grid, dim3(256), 0, st, cent, c3, norms, redo, s.n, ntile, tiles);
    else hipLaunchKernelGGL(split3_kernel<128>, grid, dim3(256), 0, st, cent, c3, norms, redo, s.n, ntile, tiles);
    return hipGetLastError();
}

template <int D, int TA>
static hipError_t few_launch(const Dims& s, const void* Q, const bf16_t* c3, int32_t* idx, hipStream_t st)
{
    const int strips = (s.N + 15) / 16;
    const size_t lds = sizeof(uint32_t) * (size_t)kGateWaves * select_words<TA>(s.k);
    hipError_t e = ensure_dynamic_lds((const void*)gate_few_kernel<D, TA>, lds);
    if (e != hipSuccess) return e;
    ProfileScope timing(MOBA_PROFILE_TOPK, st);
    hipLaunchKernelGGL((gate_few_kernel<D, TA>), dim3((unsigned)schedule_grid(s.bh, (strips + kGateWaves - 1) / kGateWaves)),
                       dim3(kGateWaves * kWave), lds, st, (const bf16_t*)Q, c3, (s.n + 15) / 16, idx, s.N, s.B, s.k, strips,
                       s.bh, s.G, s.blk_first);
    return hipGetLastError();
}

template <int D, int KC>
static hipError_t many_launch(const Dims& s, const void* Q, const bf16_t* c3, const float4* norms,
                              int32_t* redo, int32_t* idx, hipStream_t st)
{
    // one sequence: its first queries have few candidates, the rest many; packed batches: either anywhere
    constexpr int kRows = 16 * GateCfg<KC>::QT;
    const int64_t border = s.blk_first ? 0 : (int64_t)16 * kGateFew<D> * s.B, few_end = s.blk_first ? s.N : std::min<int64_t>(s.N, border + s.B);
    const int strips = (s.N + kRows - 1) / kRows, few_strips = (int)((few_end + 15) / 16);
    const int many_wgs = (int)((strips - border / kRows + kGateWaves - 1) / kGateWaves);
    const int few_wgs = (few_strips + kGateWaves - 1) / kGateWaves;
    const size_t lds = sizeof(uint32_t) * (size_t)kGateWaves * GateLds<KC>::WORDS;
    hipError_t e = ensure_dynamic_lds((const void*)gate_many_kernel<D, KC>, lds);
    if (e != hipSuccess) return e;
    ProfileScope timing(MOBA_PROFILE_TOPK, st);
    hipLaunchKernelGGL((gate_many_kernel<D, KC>), dim3((unsigned)schedule_grid(s.bh, many_wgs + few_wgs)),
                       dim3(kGateWaves * kWave), lds, st, (const bf16_t*)Q, c3, norms, (s.n + 15) / 16, idx, redo, s.N,
                       s.B, s.n, s.k, strips, many_wgs, few_strips, few_wgs, s.bh, s.G, s.blk_first);
    return hipGetLastError();
}

hipError_t launch_gate(const Dims& s, const void* Q, const float* cent, int32_t* idx, void* ws, hipStream_t st)
{
    if (s.bh == 0 || s.N == 0) return hipSuccess;
    if (s.dtype != MOBA_BF16) {
        const int strips = (s.N + 15) / 16;
        const dim3 grid((unsigned)schedule_grid(s.bh, (strips + kGateWaves - 1) / kGateWaves));
        const size_t lds = sizeof(uint32_t) * (size_t)kGateWaves * select_words<kGateF32Tiles>(s.k);
        if (s.D == 64)
            hipLaunchKernelGGL(gate_f32_kernel<64>, grid, dim3(kGateWaves * kWave), lds, st, (const float*)Q, cent, idx, s.N,
                               s.B, s.n, s.k, strips, s.bh, s.G, s.blk_first);
        else
            hipLaunchKernelGGL(gate_f32_kernel<128>, grid, dim3(kGateWaves * kWave), lds, st, (const float*)Q, cent, idx, s.N,
                               s.B, s.n, s.k, strips, s.bh, s.G, s.blk_first);
        return hipGetLastError();
    }
    char* p = static_cast<char*>(ws);
    bf16_t* c3 = reinterpret_cast<bf16_t*>(p);
    const bool may = gate_may_redo(s);
    float4* norms = may ? reinterpret_cast<float4*>(p + terms_bytes(s)) : nullptr;
    int32_t* redo = may ? reinterpret_cast<int32_t*>(p + terms_bytes(s) + norms_bytes(s)) : nullptr;
    hipError_t e = launch_split3(s, cent, c3, norms, redo, st);
    if (e != hipSuccess) return e;
    if (!may)
        return s.D == 128 ? few_launch<128, kGateFew<128>>(s, Q, c3, idx, st)
                          : few_launch<64, kGateFew<64>>(s, Q, c3, idx, st);
    e = s.D == 64 ? many_launch<64, 8>(s, Q, c3, norms, redo, idx, st)
        : s.k <= 8 ? many_launch<128, 8>(s, Q, c3, norms, redo, idx, st)
                    : many_launch<128, 32>(s, Q, c3, norms, redo, idx, st);
    if (e != hipSuccess) return e;
    return launch_topk_redo(s, Q, c3, redo, idx, st);
}

}  // namespace moba
