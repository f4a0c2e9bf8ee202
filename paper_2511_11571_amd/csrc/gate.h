// Selection helpers of the gate kernels: the scores of 16 queries live in the registers of one wave,
// four lanes (16 g + m16, g = 0 .. 3) per query.
#pragma once
#include "mfma.h"

namespace moba {

constexpr float kFltMax = 3.402823466e+38f;
constexpr float kScoreMax = 1e38f;           // scores held in registers are clamped to +-this (a NaN to the largest)

template <typename F>
__device__ __forceinline__ uint32_t over_g_bits(uint32_t x, F f)       // f over the four lanes of a query, in all of them
{
    const auto h = __builtin_amdgcn_permlane32_swap(x, x, false, false);
    const uint32_t y = f(h[0], h[1]);
    const auto q = __builtin_amdgcn_permlane16_swap(y, y, false, false);
    return f(q[0], q[1]);
}
__device__ __forceinline__ int sum_g(int x)
{
    return (int)over_g_bits((uint32_t)x, [](uint32_t a, uint32_t b) { return a + b; });
}
__device__ __forceinline__ uint32_t or_g(uint32_t x)
{
    return over_g_bits(x, [](uint32_t a, uint32_t b) { return a | b; });
}
__device__ __forceinline__ float fsum_g(float x)
{
    return __uint_as_float(over_g_bits(__float_as_uint(x), [](uint32_t a, uint32_t b) {
        return __float_as_uint(__uint_as_float(a) + __uint_as_float(b));
    }));
}
__device__ __forceinline__ float fmax_g(float x)
{
    return __uint_as_float(over_g_bits(__float_as_uint(x), [](uint32_t a, uint32_t b) {
        return __float_as_uint(fmaxf(__uint_as_float(a), __uint_as_float(b)));
    }));
}
__device__ __forceinline__ float fmin_g(float x) { return -fmax_g(-x); }
__device__ __forceinline__ uint32_t umax_g(uint32_t x)
{
    return over_g_bits(x, [](uint32_t a, uint32_t b) { return a > b ? a : b; });
}
__device__ __forceinline__ uint32_t umin_g(uint32_t x)
{
    return over_g_bits(x, [](uint32_t a, uint32_t b) { return a < b ? a : b; });
}

// ---- threshold search.  c(t) = number of a query's values >= t.  A bracket [lo, hi) is kept with
// c(lo) = clo >= need and c(hi) = chi < need; a probe is placed by interpolating log c between its ends
// (score distributions have tails that fall off much like that), aimed a few counts to the side of the
// end that is further away so that both ends move; every fifth probe halves the bracket, which bounds the
// number of probes whatever the distribution.  The sixteen queries of a wave search side by side.
struct Bracket {
    int clo, chi;
    int lane_lo = 0, lane_hi = 0;        // this lane's part of both
};

// where to probe, as a fraction of the bracket
__device__ __forceinline__ float probe(int need, int slack, const Bracket& b, int it)
{
    if (it % 5 == 4) return 0.5f;
    const float width = (float)(b.clo - b.chi);
    const float aside = width <= 6.f ? 0.f : fminf(5.6f, 0.3f * width);
    float aim = (float)need + 0.5f * (float)slack + (b.clo - need > need - b.chi ? aside : -aside);
    aim = fminf(fmaxf(aim, (float)b.chi + 0.5f), (float)b.clo - 0.5f);
    const float top = fast_log2((float)b.clo + 0.5f);
    return (top - fast_log2(aim)) * __builtin_amdgcn_rcpf(top - fast_log2((float)b.chi + 0.5f));
}

// standard normal quantile: z with P(Z >= z) = p, absolute error below 5e-4 (Abramowitz and Stegun
// 26.2.23); only ever a first guess
__device__ __forceinline__ float normal_quantile(float p)
{
    const float q = fminf(p, 1.f - p);
    const float t = sqrtf(fmaxf(-2.f * kLn2 * fast_log2(fmaxf(q, 1e-30f)), 0.f));
    const float z = t - (2.515517f + t * (0.802853f + t * 0.010328f)) *
                            __builtin_amdgcn_rcpf(1.f + t * (1.432788f + t * (0.189269f + t * 0.001308f)));
    return p < 0.5f ? z : -z;
}

// scores x[0 .. NX) of a lane, of which the first `used` (the same in all lanes) are set and the rest is -inf
template <int NX>
__device__ __forceinline__ int count_lane(const f32x4_t (&x)[NX], int used, float t)
{
    int c = 0;
#pragma unroll
    for (int u = 0; u < NX; u += 4)
        if (u < used) {                                      // (no break: the loop has to unroll, x lives in registers)
#pragma unroll
            for (int v = 0; v < 4; ++v)
                if (u + v < NX) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) c += (int)(x[u + v][i] >= t);
                }
        }
    return c;
}

// until need <= clo <= need + slack or at most `few` values are left in the bracket, or no number lies
// inside it (its values are equal).  On entry c(lo) = b.clo >= need and nothing reaches hi; `first`: the
// first probe (NAN: none).
template <int NX>
__device__ __forceinline__ void search_threshold(const f32x4_t (&x)[NX], int used, int need, int slack, int few,
                                                 float first, float& lo, float& hi, Bracket& b)
{
    b.chi = 0;
    bool stuck = false;
    for (int it = 0;; ++it) {
        const bool act = b.clo > need + slack && b.clo - b.chi > few && !stuck;
        if (!__ballot(act)) break;
        const float mid = 0.5f * lo + 0.5f * hi;
        float t = it == 0 && first == first ? first : lo + (hi - lo) * probe(need, slack, b, it);
        if (!(t > lo && t < hi)) t = mid;
        stuck = stuck || (act && !(t > lo && t < hi));
        const int mine = count_lane<NX>(x, used, t), c = sum_g(mine);
        if (act && !stuck) {
            if (c >= need) { lo = t; b.clo = c; b.lane_lo = mine; }
            else { hi = t; b.chi = c; b.lane_hi = mine; }
        }
    }
}

// the same for distinct unsigned keys y (0: none): afterwards exactly `need` keys are >= the result
template <int NY>
__device__ __forceinline__ uint32_t search_key(const uint32_t (&y)[NY], uint32_t lo, uint32_t hi, int need, int total)
{
    Bracket b = {total, 0};
    for (int it = 0;; ++it) {
        const bool act = b.clo > need && hi - lo > 1u;
        if (!__ballot(act)) break;
        const uint32_t span = hi - lo;
        const uint32_t step = min((uint32_t)((float)span * probe(need, 0, b, it)), span - 1u);
        const uint32_t t = lo + max(step, 1u);
        int c = 0;
#pragma unroll
        for (int j = 0; j < NY; ++j) c += (int)(y[j] >= t);
        c = sum_g(c);
        if (act) {
            if (c >= need) { lo = t; b.clo = c; }
            else { hi = t; b.chi = c; }
        }
    }
    return lo;
}

// Rows of topk_idx out of LDS: stage[q][k + 1] -> out[q][k], q = 0 .. nq - 1, one wave, consecutive
// 4-byte stores
__device__ __forceinline__ void store_rows(const int32_t* stage, int32_t* __restrict__ out, int nq, int k, int lane)
{
    const int total = nq * k;
    const int dq = kWave / k, dp = kWave % k;
    int q = lane / k, p = lane % k;
    for (int i = lane; i < total; i += kWave) {
        out[i] = stage[q * (k + 1) + p];
        q += dq;
        p += dp;
        if (p >= k) { p -= k; ++q; }
    }
}

// Bit rows (row q of Wn words, queries b0 .. b0 + batch - 1 of the 16) -> ascending block ids in
// stage[q][k + 1], by the four lanes of each query; `here`: this lane's query is one of them
__device__ __forceinline__ void rows_from_bits(const uint32_t* row, int Wn, bool here, int first_block, int k,
                                               int32_t* stage_row, int lane)
{
    const int m16 = lane & 15, g = lane >> 4;
    const int wq = (Wn + 3) / 4, w0 = min(Wn, g * wq), w1 = min(Wn, w0 + wq);
    int mine = 0;
    if (here) {
#pragma unroll 8
        for (int w = w0; w < w1; ++w) mine += __popc(row[w]);
    }
    // entries of the lanes g' < g
    const int c0 = __shfl(mine, m16, kWave), c1 = __shfl(mine, m16 + 16, kWave), c2 = __shfl(mine, m16 + 32, kWave);
    int p = (g > 0 ? c0 : 0) + (g > 1 ? c1 : 0) + (g > 2 ? c2 : 0);
    if (here) {
        uint32_t next = w0 < w1 ? row[w0] : 0u;
        for (int w = w0; w < w1; ++w) {
            uint32_t word = next;
            next = row[min(w + 1, w1 - 1)];
            while (word) {
                if (p < k) stage_row[p] = first_block + 32 * w + __ffs(word) - 1;
                ++p;
                word &= word - 1u;
            }
        }
        // the last lane fills the row up
        if (g == 3)
            for (; p < k; ++p) stage_row[p] = -1;
    }
}

constexpr int kFew = 14;                  // values that the last step ranks directly
constexpr int kFewSlots = 16;

// LDS words of a wave for select_and_stage
template <int NX>
constexpr int select_words(int k) { return 16 * (k + 1) + 16 * (NX / 2) + 16 * 2 * kFewSlots; }

// largest, smallest, sum and sum of squares of a lane's scores; fold(): four more of them, of which those
// outside [0, count) -- place0 + i -- are no candidates
struct ScoreStats {
    float mx = -INFINITY, mn = INFINITY, sum = 0.f, sq = 0.f;
    __device__ __forceinline__ void fold(const f32x4_t& sc, f32x4_t& x, bool edge, int place0, int count)
    {
        if (!edge) {                                         // (maxima that hand a NaN on)
            mx = max_nan(max_nan(max_nan(sc[0], sc[1]), sc[2]), max_nan(sc[3], mx));
            mn = min_nan(min_nan(min_nan(sc[0], sc[1]), sc[2]), min_nan(sc[3], mn));
#pragma unroll
            for (int i = 0; i < 4; ++i) { sum += sc[i]; sq = fmaf(sc[i], sc[i], sq); }
            x = sc;
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const bool in = (uint32_t)(place0 + i) < (uint32_t)count;
                const float w = in ? sc[i] : 0.f;
                x[i] = in ? sc[i] : -INFINITY;
                mx = max_nan(mx, x[i]);
                mn = min_nan(mn, in ? sc[i] : INFINITY);
                sum += w;
                sq = fmaf(w, w, sq);
            }
        }
    }
    __device__ __forceinline__ static float min_nan(float a, float b) { return __builtin_elementwise_minimum(a, b); }
    // scores that are no numbers, or so large that differences overflow: clamped to +-kScoreMax (a NaN to
    // the largest); -inf marks what is no candidate (an edge's), which `count` of them tells apart
    template <int NX>
    __device__ __forceinline__ void tame(f32x4_t (&x)[NX], int used, int place0, int count)
    {
        if (!__ballot(!(mx < kScoreMax && (mn > -kScoreMax)))) return;
        mx = -INFINITY; mn = INFINITY; sum = 0.f; sq = 0.f;
#pragma unroll
        for (int u = 0; u < NX; ++u)
            if (u < used) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const bool in = (uint32_t)(place0 + 16 * u + i) < (uint32_t)count;
                    x[u][i] = in ? fmaxf(fminf(x[u][i], kScoreMax), -kScoreMax) : -INFINITY;
                    mx = fmaxf(mx, x[u][i]);
                    mn = fminf(mn, in ? x[u][i] : INFINITY);
                }
            }
        if (mn == INFINITY) mn = 0.f;
    }
};

// Selection of one 16-query group whose scores are all in registers (x[u][i]: block 16 (tbeg + u) + 4 g + i,
// -inf where that is no candidate): exact, ties to the lower block; kept blocks ascending to
// stage[q][k + 1], stage = lds.  About four probes over the registers (the first from mean and variance)
// leave at most 14 scores between the ends of the bracket; those are filed in LDS and ranked by the
// query's four lanes, and one more pass turns everything from the bracket's upper end on into places.
// Nothing in it waits for an LDS atomic: a lane knows from the counts where its scores go.
template <int NX>
__device__ __forceinline__ void select_and_stage(f32x4_t (&x)[NX], const ScoreStats& st, int used, int tbeg, int need,
                                                 int past, int k, uint32_t* lds, int lane)
{
    const int m16 = lane & 15, g = lane >> 4;
    int32_t* row = reinterpret_cast<int32_t*>(lds) + m16 * (k + 1);
    uint32_t* chosen = lds + 16 * (k + 1);                   // [NX / 2][16]: kept ones among the filed scores, 32 blocks a word
    // [16][kFewSlots] scores, then as many block numbers (apart: a score and its number side by side would
    // be stored as one 64-bit register pair, and every score of x would take two registers)
    uint32_t* few = chosen + 16 * (NX / 2);
    uint32_t* few_blk = few + 16 * kFewSlots;
    float lo = fmin_g(st.mn), hi = fmax_g(st.mx);
    hi += fabsf(hi) * 1e-6f + 1e-30f;                        // above every score
    Bracket b = {need > 0 ? past : 0, 0};
    b.lane_lo = count_lane<NX>(x, used, lo);
    {
        const float inv = 1.f / (float)max(past, 1), mean = fsum_g(st.sum) * inv;
        const float var = fmaxf(fsum_g(st.sq) * inv - mean * mean, 0.f);
        search_threshold<NX>(x, used, need, 0, kFew, mean + sqrtf(var) * normal_quantile((float)need * inv), lo, hi, b);
    }
    // the bracket is beyond doubt (clo == need: keep from lo on), or holds a few scores to rank, or -- more
    // than kFew equal ones -- ties
    const bool rank = b.clo > need && b.clo - b.chi <= kFew, ties = b.clo > need && !rank;
    const float sure = b.clo > need ? hi : need > 0 ? lo : INFINITY;
    for (int i = lane; i < 16 * (NX / 2); i += kWave) chosen[i] = 0u;
    if (__ballot(rank)) {
        const float from = rank ? lo : INFINITY;
        const int mine = rank ? b.lane_lo - b.lane_hi : 0;
        // scores filed by the lanes g' < g of the query
        const int c0 = __shfl(mine, m16, kWave), c1 = __shfl(mine, m16 + 16, kWave), c2 = __shfl(mine, m16 + 32, kWave);
        const int c3 = __shfl(mine, m16 + 48, kWave), c = c0 + c1 + c2 + c3;
        uint32_t* at = few + m16 * kFewSlots + (g > 0 ? c0 : 0) + (g > 1 ? c1 : 0) + (g > 2 ? c2 : 0);
#pragma unroll
        for (int u = 0; u < NX; ++u)
            if (u < used) {
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (x[u][i] >= from && x[u][i] < hi) {
                        at[0] = __float_as_uint(x[u][i]);
                        at[16 * kFewSlots] = 16 * u + i;     // (+ 4 g: by the reader, from the place)
                        ++at;
                    }
            }
        __builtin_amdgcn_wave_barrier();
        // (the places say which lane filed a score: 4 g of its block number)
        auto owner = [&](int e) { return 4u * ((uint32_t)(e >= c0) + (uint32_t)(e >= c0 + c1) + (uint32_t)(e >= c0 + c1 + c2)); };
        // each lane takes every fourth of them; all in registers: one LDS latency
        uint64_t v[kFewSlots];
        const uint4* scores = reinterpret_cast<const uint4*>(few + m16 * kFewSlots);
        const uint4* blocks = reinterpret_cast<const uint4*>(few_blk + m16 * kFewSlots);
#pragma unroll
        for (int e = 0; e < kFewSlots; e += 4) {
            const uint4 a = scores[e / 4], d = blocks[e / 4];
            const uint32_t sv[4] = {a.x, a.y, a.z, a.w}, bv[4] = {d.x, d.y, d.z, d.w};
#pragma unroll
            for (int h = 0; h < 4; ++h)                      // (score, then lower block first) as one number: larger = better
                v[e + h] = e + h < c ? ((uint64_t)order_key(__uint_as_float(sv[h])) << 32) | (uint32_t)~(bv[h] + owner(e + h)) : 0u;
        }
        const int want = need - b.chi;
#pragma unroll
        for (int a = 0; a < kFewSlots; a += 4) {
            uint64_t me = v[a];
#pragma unroll
            for (int o = 1; o < 4; ++o) me = g == o ? v[a + o] : me;
            int above = 0;
#pragma unroll
            for (int o = 0; o < kFewSlots; ++o) above += (int)(v[o] > me);
            const uint32_t blk = ~(uint32_t)me;
            if (a + g < c && above < want && rank) atomicOr(&chosen[(blk >> 5) * 16 + m16], 1u << (blk & 31));
        }
    }
    if (__ballot(ties)) {
        // equal scores: the lowest blocks among them, one after the other
        int left = ties ? need - b.chi : 0;
        uint32_t last = 0u;                                  // blocks below this one are taken
        while (__ballot(left > 0)) {
            uint32_t best = 0xffffffffu;
            asm volatile("" : "+v"(lo), "+v"(hi));           // (or the compares would be hoisted out of the loop and spill)
            const int from = (int)last - 4 * g;              // (block numbers as constants, for the same reason)
#pragma unroll
            for (int u = 0; u < NX; ++u)
                if (u < used) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const bool in = x[u][i] >= lo && x[u][i] < hi && 16 * u + i >= from;
                        best = in ? min(best, (uint32_t)(16 * u + i)) : best;
                    }
                }
            best = umin_g(best == 0xffffffffu ? best : best + 4 * g);
            if (left > 0 && best != 0xffffffffu) {
                if (g == 0) atomicOr(&chosen[(best >> 5) * 16 + m16], 1u << (best & 31));
                last = best + 1u;
            }
            --left;
        }
    }
    __builtin_amdgcn_wave_barrier();
    // ascending rows: two tiles (32 blocks) at a time as one word in all four lanes of the query; a lane
    // writes its own eight blocks at base + the number of kept ones before them
    int base = 0;
    uint32_t extra[NX / 2];
#pragma unroll
    for (int u = 0; u < NX / 2; ++u) extra[u] = 2 * u < used ? chosen[u * 16 + m16] : 0u;
#pragma unroll
    for (int u = 0; u < NX; u += 2)
        if (u < used) {
            uint32_t w = 0;
#pragma unroll
            for (int v = 0; v < 2; ++v)
#pragma unroll
                for (int i = 0; i < 4; ++i) w |= x[u + v][i] >= sure ? 1u << (16 * v + i) : 0u;
            w = or_g(w << (4 * g)) | extra[u / 2];
            const uint32_t mine = w >> (4 * g);
#pragma unroll
            for (int v = 0; v < 2; ++v)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int bit = 16 * v + i;
                    if ((mine >> bit) & 1u) {
                        const int p = base + __popc(w & ((1u << (bit + 4 * g)) - 1u));
                        if (p < k) row[p] = 16 * (tbeg + u) + bit + 4 * g;
                    }
                }
            base += __popc(w);
        }
    for (int p = base + g; p < k; p += 4) row[p] = -1;
    __builtin_amdgcn_wave_barrier();
}

}  // namespace moba
