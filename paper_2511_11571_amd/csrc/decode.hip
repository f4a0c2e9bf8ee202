// Decode-shaped MoBA forward (inference): the last q_len positions of a sequence of N keys, each
// query routed and attended on its own -- the operator of the paper's Section 2 for a few query
// rows and a long key sequence, where N need not be a multiple of the block size: a query's own
// block is then the ragged last block, attended causally like any own block (the centroid
// algorithm of Appendix C.1 treats the tail block the same way; here its centroid is never
// needed, because the own block is not a routing candidate).
//
// One workgroup of 16 waves per (query, batch*head) (or a few, see decode_splits()): gate scores against the centroids
// of the complete past blocks, exact top-k, attention over the kept blocks and the own block, all in
// fp32 arithmetic; nothing is written to global memory but O, lse, (optionally) the kept blocks and the parts of shared queries.
//
// The work per query is a few hundred KB of reads from a chip that is mostly idle, so the kernel is
// bound by how fast ONE compute unit takes them in and by the chain of dependent steps:
//  - every read of centroids, K and V covers whole rows with neighbouring lanes (16 bytes each): a
//    lane per row moves a quarter of the bytes per clock on this chip.  The lanes of a row add their
//    parts of the dot product up by DPP;
//  - the keys of all kept blocks and the own block count as ONE sequence that the waves walk together:
//    with a block per wave, 9 kept blocks left 7 of 16 waves idle;
//  - loads go out in batches of 16 per lane (a batch is one memory latency), the last one smaller;
//  - every group of lanes that holds a key keeps a softmax of its own (m, l, O), merged once at the
//    end: no cross-lane maximum or sum inside the walk;
//  - the selection of up to 16 blocks takes a lower bound of the k-th largest score from the maxima of 64 groups and
//    ranks the few scores that reach it, sixteen lanes per score (three barriers, 2.9 -> 1.6 us at k = 8 of 1024).  Longer rows, and
//    calls where too many scores reach the bound, bin the scores linearly between the smallest and the largest (1024 bins, one LDS
//    atomic per score, well spread), and rank only the scores of the bin that holds the k-th largest;
//    the radix select over the bits of the scores remains for bins of more than 128 scores (ties, or one
//    score far from the rest) and for non-finite scores;
//  - queries that share a key/value head run on the same XCD at the same time (schedule()).
// Of 12.3 us inside one workgroup (1 query of 131109 keys, d = 64, B = 128, k = 8; binned selection) the gate took 4.2, the selection
// 2.9, the keys 4.5 and the merge 0.7; both memory phases (262 and 272 KB) run at the 25 bytes per clock one compute unit takes in here.
// 1 query of 131109 keys x 32 slices: 24.8 -> 13.1 -> 11.5 us (the kernel alone 11.1; a call takes the host 9 to 10); 16 queries of 32805
// keys x 16 heads on 4 key/value heads (d = 128, B = 64, k = 32): 59 -> 27.7 -> 26.3 us (there
// 340 MB go from the L2s to the compute units and 126 MB from behind them: 5 TB/s of the latter).
#include <algorithm>
#include <atomic>
#include <chrono>
#include <type_traits>

#include "common.h"

namespace moba {

// fp32 -> uint32 with the same order (negative numbers reversed, then below the positive ones)
__device__ __forceinline__ uint32_t decode_key(float x)
{
    const uint32_t b = __float_as_uint(x);
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

template <int CTRL, int ROWS = 0xf, typename X>
__device__ __forceinline__ X dpp(X v)                        // lanes without a source (or outside ROWS) read 0
{
    static_assert(sizeof(X) == 4, "32-bit values");
    const int r = __builtin_amdgcn_update_dpp(0, *reinterpret_cast<const int*>(&v), CTRL, ROWS, 0xf, true);
    return *reinterpret_cast<const X*>(&r);
}

// sum over the L (8, 16 or 32) neighbouring lanes of a row, in all of them
template <int L>
__device__ __forceinline__ float row_sum(float x)
{
    x += dpp<0xb1>(x);                                       // quad_perm 1,0,3,2
    x += dpp<0x4e>(x);                                       // quad_perm 2,3,0,1
    x += dpp<0x141>(x);                                      // row_half_mirror: the other quad of 8
    if constexpr (L >= 16) x += dpp<0x140>(x);               // row_mirror: the other half of 16
    if constexpr (L >= 32) {
        const uint32_t b = __float_as_uint(x);
        const auto q = __builtin_amdgcn_permlane16_swap(b, b, false, false);
        x = __uint_as_float(q[0]) + __uint_as_float(q[1]);
    }
    return x;
}

// sum of the counts of 16 neighbouring lanes, in all of them
__device__ __forceinline__ int count_16(int x)
{
    x += dpp<0xb1>(x);
    x += dpp<0x4e>(x);
    x += dpp<0x141>(x);
    x += dpp<0x140>(x);
    return x;
}

// f over the lanes that are a multiple of L apart, in all of them (all lanes of a row of L agree or
// hold different channels): the other half of a 16-lane row by DPP, the rest by lane swaps
template <int L, typename F>
__device__ __forceinline__ float across_rows(float x, F f)
{
    if constexpr (L <= 8) x = f(x, dpp<0x128>(x));           // row_ror 8
    if constexpr (L <= 16) {
        const uint32_t b = __float_as_uint(x);
        const auto q = __builtin_amdgcn_permlane16_swap(b, b, false, false);
        x = f(__uint_as_float(q[0]), __uint_as_float(q[1]));
    }
    const uint32_t b = __float_as_uint(x);
    const auto h = __builtin_amdgcn_permlane32_swap(b, b, false, false);
    return f(__uint_as_float(h[0]), __uint_as_float(h[1]));
}

// a + the two products of bf16 pairs
__device__ __forceinline__ float dot2(uint32_t x, uint32_t y, float a)
{
    typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
    return __builtin_amdgcn_fdot2_f32_bf16(*reinterpret_cast<bf16x2_t*>(&x), *reinterpret_cast<bf16x2_t*>(&y), a, false);
}

// inclusive prefix sum over the 64 lanes of a wave
__device__ __forceinline__ int wave_prefix(int x)
{
    x += dpp<0x111>(x);                                      // row_shr 1, 2, 4, 8: inside rows of 16
    x += dpp<0x112>(x);
    x += dpp<0x114>(x);
    x += dpp<0x118>(x);
    x += dpp<0x142, 0xa>(x);                                 // row_bcast 15: rows 1 and 3 take the row before
    x += dpp<0x143, 0xc>(x);                                 // row_bcast 31: rows 2 and 3 take the lower half
    return x;
}

constexpr int kDecodeWaves = 16;
constexpr int kDecodeThreads = kDecodeWaves * kWave;
constexpr int kDecodeBins = kDecodeThreads;    // bins of the selection: one per thread
// Most scores of one bin that are ranked directly.  Each of them meets all the others, the radix select takes the
// same time for any number: a score 10000 times the rest puts those into one bin (1 query, 1024 blocks, k = 8, whole call:
// 52.0 us ranked, 17.8 by the radix select).
constexpr int kDecodeRank = 128;
// Rows up to this length are selected from the scores that reach a bound taken from the maxima of kDecodeGroups groups: of n
// scores about n (1 - (1 - k / groups)^(groups / n)), 11 of 1024 at k = 8 and 90 of 4096 at k = 48.  Longer rows gain nothing or
// lose (whole call, bins -> bound: k = 8 of 140 blocks 24.0 -> 22.0 us, 16 of 35 17.1 -> 17.6, 24 of 3750 17.0 -> 16.8, 30 of 140 12.8
// -> 12.6, 40 of 1875 13.8 -> 14.9, 48 of 3750 18.4 -> 20.2).
constexpr int kDecodeShort = 16;
constexpr int kDecodeGroups = 4 * kDecodeWaves;
static_assert(kDecodeGroups == kWave, "a group's maximum per lane");
constexpr int kDecodeBoundBit = 18;            // the bound's lowest bit (5 bits of a score's fraction: a few scores more)
// words that hold the ranked scores, then the waves' (m, l, O)
template <int D>
constexpr int kDecodeScratch = 2 * kDecodeRank > kDecodeWaves * (D + 2) ? 2 * kDecodeRank : kDecodeWaves * (D + 2);

constexpr int kDecodeSplits = 8;               // most workgroups that share a query
// Several workgroups per query: what they share
struct DecodeSplit {
    uint64_t* arrived;                          // [queries]
    float* part;                                // [queries][splits][m, l, O]
    uint64_t tag;
};

// SHARED: several workgroups per query.  SHORT: rows of up to kDecodeShort kept blocks.  Instantiations of their own: in one, calls of
// longer rows that nobody shares paid for registers and code of both (graph of calls, us, one kernel -> four: 60 queries, d = 64, B = 32,
// k = 29 of 48 blocks 11.40 -> 11.24, 60 of B = 64 14.78 -> 14.64, as before either was there: 11.27, 14.64).
template <typename T, int D, bool SHARED, bool SHORT>
__global__ __launch_bounds__(kDecodeThreads) void decode_kernel(
    const T* __restrict__ Q, const T* __restrict__ K, const T* __restrict__ V,
    const float* __restrict__ cent, T* __restrict__ O, float* __restrict__ lse,
    int32_t* __restrict__ idx_out, int N, int B, int k, int q_len, int cblocks, float scale, int G,
    int bhk, int npast_max, int shares, DecodeSplit split)
{
    const int splits = SHARED ? shares : 1;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    constexpr int NT = kDecodeThreads, NW = kDecodeWaves;
    constexpr int LPR = D * (int)sizeof(T) / 16;            // lanes of a K / V row, 16 bytes each
    constexpr int EPL = 16 / (int)sizeof(T);                // elements of a lane
    constexpr int RPI = kWave / LPR;                        // rows per load instruction of a wave
    float* sc = reinterpret_cast<float*>(smem_raw);         // [npast_max rounded up to 4] gate scores
    uint32_t* hist = reinterpret_cast<uint32_t*>(sc + (npast_max + 3) / 4 * 4);   // [kDecodeBins]
    uint2* cand = reinterpret_cast<uint2*>(hist + kDecodeBins);                   // [kDecodeRank] scores to rank: (key, block) or, as one 64-bit number, (key, ~block)
    float* mrg = reinterpret_cast<float*>(cand);            // [NW][D + 2] the waves' (m, l, O), after the selection
    uint32_t* keep = reinterpret_cast<uint32_t*>(mrg + kDecodeScratch<D>);        // kept-block bits of the ranked bin
    float* wmx = reinterpret_cast<float*>(keep + (npast_max + 31) / 32);          // [NW] and
    float* wmn = wmx + NW;                                  // [NW]: the waves' largest and smallest score
    int* wcnt = reinterpret_cast<int*>(wmn + NW);           // [NW]
    int* ctl = wcnt + NW;                                   // [5]
    uint32_t* gmx = reinterpret_cast<uint32_t*>(ctl + 5);   // [kDecodeGroups] order-preserving keys of the groups' largest scores
    int* sel = ctl + 5 + kDecodeGroups;                     // [k + 1] kept blocks, ascending, then the own block

    const int tid = threadIdx.x, lane = tid % kWave;
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    int skv, pos;
    if (!schedule(blockIdx.x, bhk, G * q_len * splits, skv, pos)) return;
    const int share = SHARED ? pos % splits : 0;        // this workgroup's share of the query's keys
    if (SHARED) pos /= splits;
    const int s = skv * G + pos / q_len, r = pos % q_len;   // G query heads share a key/value head
    const int t = N - q_len + r;                            // position of the query
    const int past = t / B;                                 // complete blocks before its own block
    const int64_t qrow = (int64_t)s * q_len + r;

    // the lane's pieces of the query, for the gate (channels 64 c + 4 (lane mod 16) ..) and for q . k
    const int piece = lane % LPR, kslot = lane / LPR;
    const float c2 = scale * 1.4426950408889634f;           // logits in log2 units
    uint32_t qb[4];
    {
        const uint4 x = *reinterpret_cast<const uint4*>(Q + qrow * D + piece * EPL);
        qb[0] = x.x; qb[1] = x.y; qb[2] = x.z; qb[3] = x.w;
    }
    hist[tid] = 0u;
    for (int i = tid; i < (past + 31) / 32; i += NT) keep[i] = 0u;
    if (tid < 5) ctl[tid] = 0;

    const int want = min(k, past);
    if (past > k && k > 0) {
        // ---- gate scores q . centroid_j: 16 lanes per centroid, D / 16 channels each
        {
            constexpr int CL = D / 64;                      // 16-byte loads per lane and row
            const int cl = lane & 15, cr = lane >> 4;
            float4 q4[CL];
#pragma unroll
            for (int c = 0; c < CL; ++c) {
                const T* qc = Q + qrow * D + 64 * c + 4 * cl;
                if constexpr (sizeof(T) == 2) {
                    const uint2 x = *reinterpret_cast<const uint2*>(qc);
                    q4[c] = make_float4(__uint_as_float(x.x << 16), __uint_as_float(x.x & 0xffff0000u),
                                        __uint_as_float(x.y << 16), __uint_as_float(x.y & 0xffff0000u));
                } else {
                    q4[c] = *reinterpret_cast<const float4*>(qc);
                }
            }
            const char* cs = reinterpret_cast<const char*>(cent + (int64_t)skv * cblocks * D);
            float mx = -INFINITY, mn = INFINITY;
            constexpr int U = 16 / CL;                      // rows in flight per lane group
            constexpr uint32_t ROW = D * sizeof(float);
            for (int j0 = 4 * wave; j0 < past; j0 += 4 * NW * U) {
                float4 x[U][CL];
#pragma unroll
                for (int u = 0; u < U; ++u) {               // (past the end: the last row again, dropped)
                    const int first = min(j0 + 4 * NW * u, past - 1);               // the same in all lanes
                    const char* row = cs + (int64_t)first * ROW;
                    const uint32_t o = (uint32_t)min(cr, past - 1 - first) * ROW + 16u * cl;
#pragma unroll
                    for (int c = 0; c < CL; ++c) x[u][c] = *reinterpret_cast<const float4*>(row + o + 256 * c);
                }
                float mine = 0.f;                           // lane cl of a group keeps the score of row u = cl
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    float a = 0.f;
#pragma unroll
                    for (int c = 0; c < CL; ++c) {
                        a = fmaf(x[u][c].x, q4[c].x, a); a = fmaf(x[u][c].y, q4[c].y, a);
                        a = fmaf(x[u][c].z, q4[c].z, a); a = fmaf(x[u][c].w, q4[c].w, a);
                    }
                    a = row_sum<16>(a);
                    mine = cl == u ? a : mine;
                }
                const int j = j0 + 4 * NW * cl + cr;
                if (cl < U && j < past) {
                    sc[j] = mine;
                    mx = __builtin_elementwise_maximum(mx, mine);        // (hand a NaN on)
                    mn = __builtin_elementwise_minimum(mn, mine);
                }
            }
            auto fmx = [](float a, float b) { return __builtin_elementwise_maximum(a, b); };
            auto fmn = [](float a, float b) { return __builtin_elementwise_minimum(a, b); };
            mx = fmx(mx, dpp<0xb1>(mx)); mx = fmx(mx, dpp<0x4e>(mx)); mx = fmx(mx, dpp<0x141>(mx));
            if (SHORT && cl == 0) gmx[4 * wave + cr] = decode_key(fmx(mx, dpp<0x128>(mx)));   // (row_ror 8: the other half of the 16)
            mn = fmn(mn, dpp<0xb1>(mn)); mn = fmn(mn, dpp<0x4e>(mn)); mn = fmn(mn, dpp<0x141>(mn));
            mx = across_rows<8>(mx, fmx);
            mn = across_rows<8>(mn, fmn);
            if (lane == 0) { wmx[wave] = mx; wmn[wave] = mn; }
        }
        __syncthreads();
        // ---- the k largest scores, ties to the lower block (Section 2).  A thread owns up to four
        // consecutive blocks.
        // Short rows: the k-th largest of the groups' maxima (a score of its own from every group) is a lower bound of
        // the k-th largest score, and few scores reach it: those are ranked against each other.  At least k
        // of them prove the result whatever the bound.  The bound itself is searched bit by bit, by every wave for itself.
        const int j0 = 4 * tid;
        bool chosen = false;
        if constexpr (SHORT) {
            const uint32_t mine = gmx[lane];
            const float4 x = *reinterpret_cast<const float4*>(sc + min(j0, (past - 1) & ~3));
            uint32_t bound = 0;
#pragma unroll
            for (int bit = 31; bit >= kDecodeBoundBit; --bit)
                if (__popcll(__ballot(mine >= (bound | 1u << bit))) >= k) bound |= 1u << bit;
            const uint32_t key[4] = {decode_key(x.x), decode_key(x.y), decode_key(x.z), decode_key(x.w)};
            bool hit[4];
            int hits = 0;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                hit[i] = j0 + i < past && key[i] >= bound;
                hits += (int)hit[i];
            }
            if (hits > 0) {
                int at = atomicAdd(&ctl[4], hits);
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (hit[i]) {
                        if (at < kDecodeRank) cand[at] = make_uint2(~(uint32_t)(j0 + i), key[i]);
                        ++at;
                    }
            }
            __syncthreads();
            const int c = ctl[4];
            chosen = c >= k && c <= kDecodeRank;
            if (chosen) {
                // sixteen lanes per candidate: its place among them by (score, lower block first) as one number ...
                const uint64_t* all = reinterpret_cast<const uint64_t*>(cand);
                int* row = reinterpret_cast<int*>(hist);             // [k] kept blocks, best first
                for (int i = tid >> 4; i < c; i += NT / 16) {
                    const uint64_t me = all[i];
                    int r = 0;
                    for (int o = tid & 15; o < c; o += 16) r += (int)(all[o] > me);
                    r = count_16(r);
                    if ((tid & 15) == 0 && r < k) row[r] = (int)~(uint32_t)me;
                }
                __syncthreads();
                // ... and, the kept ones, in ascending order of the blocks
                const int i = tid >> 4;
                if (i < k) {
                    const int me = row[i];
                    int r = 0;
                    for (int o = tid & 15; o < k; o += 16) r += (int)(row[o] < me);
                    r = count_16(r);
                    if ((tid & 15) == 0) sel[r] = me;
                }
            }
        }
        if (!chosen) {
        // sum of the counts that the waves before this one left in wcnt
        auto waves_before = [&]() {
            return __builtin_amdgcn_readlane(wave_prefix(lane < wave ? wcnt[lane] : 0), kWave - 1);
        };
        float M = wmx[0], m = wmn[0];
#pragma unroll
        for (int w = 1; w < NW; ++w) {
            M = __builtin_elementwise_maximum(M, wmx[w]);
            m = __builtin_elementwise_minimum(m, wmn[w]);
        }
        // bin of a score: a non-decreasing function of it, so that every score of a higher bin is
        // larger than every score of a lower one
        const float inv = (float)(kDecodeBins - 1) / (M - m);
        bool direct = M - m < INFINITY && inv < INFINITY;
        float v[4];
        int bin[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            v[i] = j0 + i < past ? sc[j0 + i] : 0.f;
            bin[i] = j0 + i < past && direct ? min((int)((v[i] - m) * inv), kDecodeBins - 1) : -1;
        }
        int need = k, cut = 0;
        if (direct) {
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (bin[i] >= 0) atomicAdd(&hist[bin[i]], 1u);
            __syncthreads();
            // a thread per bin, the highest bin first: scores in the bins above it by prefix sums
            const int bin_here = kDecodeBins - 1 - tid;
            const int mine = (int)hist[bin_here];
            const int incl = wave_prefix(mine);
            if (lane == kWave - 1) wcnt[wave] = incl;
            __syncthreads();
            const int above = incl - mine + waves_before();
            if (above < k && k <= above + mine) { ctl[0] = bin_here; ctl[1] = k - above; ctl[2] = mine; }
            __syncthreads();
            cut = ctl[0];
            need = ctl[1];
            direct = ctl[2] <= kDecodeRank;                 // else: many scores close together
        }
        bool take[4];
        if (direct) {
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (bin[i] == cut) cand[atomicAdd(&ctl[3], 1)] = make_uint2(decode_key(v[i]), (uint32_t)(j0 + i));
            __syncthreads();
            const int c = ctl[3];
            if (tid < c) {
                const uint2 me = cand[tid];
                int rank = 0;
                for (int o = 0; o < c; ++o) {
                    const uint2 x = cand[o];
                    rank += (int)(x.x > me.x) | ((int)(x.x == me.x) & (int)(x.y < me.y));
                }
                if (rank < need) atomicOr(&keep[me.y >> 5], 1u << (me.y & 31));
            }
            __syncthreads();
            const uint32_t bits = j0 < past ? keep[j0 >> 5] >> (j0 & 31) : 0u;
#pragma unroll
            for (int i = 0; i < 4; ++i) take[i] = bin[i] > cut || (j0 + i < past && ((bits >> i) & 1u));
        } else {
            // radix select over the bits of the order-preserving keys, 8 bits a pass
            __syncthreads();
            if (tid == 0) { ctl[0] = 0; ctl[1] = k; }
            for (int shift = 24; shift >= 0; shift -= 8) {
                if (tid < 256) hist[tid] = 0u;
                __syncthreads();
                const uint32_t prefix = (uint32_t)ctl[0];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint32_t key = decode_key(v[i]);
                    if (j0 + i < past && (shift == 24 || (key >> (shift + 8)) == prefix))
                        atomicAdd(&hist[(key >> shift) & 255u], 1u);
                }
                __syncthreads();
                if (wave == 0) {
                    // the bin that holds the need-th largest key
                    const int left_all = ctl[1];
                    // (descending: lane l owns bins 255 - 4l .. 252 - 4l)
                    int c4[4], mine = 0;
                    const int b0 = 4 * (kWave - 1 - lane);
#pragma unroll
                    for (int i = 0; i < 4; ++i) { c4[i] = (int)hist[b0 + i]; mine += c4[i]; }
                    const int incl = wave_prefix(mine), above = incl - mine;
                    if (above < left_all && left_all <= incl) {      // (exactly one lane)
                        int left = left_all - above, b = 3;
                        for (; b > 0; --b) {
                            if (c4[b] >= left) break;
                            left -= c4[b];
                        }
                        ctl[0] = (int)((prefix << 8) | (uint32_t)(b0 + b));
                        ctl[1] = left;
                    }
                }
                __syncthreads();
            }
            // kept: keys above the k-th largest, and the first `need` blocks whose key equals it
            const uint32_t T0 = (uint32_t)ctl[0];
            need = ctl[1];
            int eq = 0;
#pragma unroll
            for (int i = 0; i < 4; ++i) eq += (int)(j0 + i < past && decode_key(v[i]) == T0);
            const int incl = wave_prefix(eq);
            if (lane == kWave - 1) wcnt[wave] = incl;
            __syncthreads();
            int before = incl - eq + waves_before();
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint32_t key = decode_key(v[i]);
                const bool tie = j0 + i < past && key == T0;
                take[i] = (j0 + i < past && key > T0) || (tie && before < need);
                before += (int)tie;
            }
            __syncthreads();
        }
        // kept blocks in ascending order: places by prefix sums over the threads
        int cnt = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) cnt += (int)take[i];
        const int incl = wave_prefix(cnt);
        if (lane == kWave - 1) wcnt[wave] = incl;
        __syncthreads();
        int place = incl - cnt + waves_before();
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (take[i] && place < k) sel[place++] = j0 + i;
        }
    } else {
        for (int j = tid; j < want; j += NT) sel[j] = j;    // no more past blocks than k: keep them all
    }
    if (tid == 0) sel[want] = past;
    __syncthreads();
    if (idx_out && share == 0)
        for (int c = tid; c < k; c += NT) idx_out[qrow * k + c] = c < want ? sel[c] : -1;

    // ---- attention over want * B + (t mod B) + 1 keys: position p is key p mod B of kept block p / B,
    // the own block last.  The waves walk the positions together, RPI positions per wave and load
    // instruction: the queries of a key/value head that run side by side on one XCD then pass the
    // same stretch of keys at about the same time and find each other's blocks in its L2.
    const int all = want * B + (t - past * B) + 1;
    const int each = SHARED ? (all + splits * RPI - 1) / (splits * RPI) * RPI : all;
    const int first = share * each, total = min(all, first + each);     // (no share is empty where queries are shared, see decode_splits(); one would weigh nothing)
    float m = -INFINITY, l = 0.f, acc[EPL];                 // log2 units
#pragma unroll
    for (int e = 0; e < EPL; ++e) acc[e] = 0.f;
    constexpr uint32_t ROWB = D * sizeof(T);
    const char* Ks = reinterpret_cast<const char*>(K) + (int64_t)skv * N * ROWB;
    const char* Vs = reinterpret_cast<const char*>(V) + (int64_t)skv * N * ROWB;
    auto widen = [](const uint4& x, float (&f)[EPL]) {
        const uint32_t w[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if constexpr (sizeof(T) == 2) {
                f[2 * i] = __uint_as_float(w[i] << 16);
                f[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
            } else {
                f[i] = __uint_as_float(w[i]);
            }
        }
    };
    // Blocks of whole load instructions (any B that is a multiple of RPI) and rows within 32 bits: the
    // RPI positions of an instruction lie in one block, so the block and the row inside it are scalars
    // that advance by additions.  Otherwise every lane divides.
    const bool whole = B % RPI == 0 && (int64_t)N * ROWB < ((int64_t)1 << 32);
    const int step_blk = NW * RPI / B, step_row = NW * RPI % B;
    int blk = (first + wave * RPI) / B, in_blk = (first + wave * RPI) % B;      // whole: the next instruction's block and row
    auto batch = [&](int p0, auto size, auto all_live, auto zeroed) {
        constexpr int NB = decltype(size)::value;           // load instructions of K (and of V) in flight
        constexpr bool ALL = decltype(all_live)::value;     // every position of the batch exists
        constexpr bool ZERO = decltype(zeroed)::value;      // values past the end count as zero
        uint4 kr[NB], vr[NB];
        // (past the end: some row that is attended anyway, weight 0)
        if (whole) {
#pragma unroll
            for (int u = 0; u < NB; ++u) {
                int row = sel[min(blk, want)] * B + in_blk + kslot;      // sel[want]: the own block
                if (!ALL) row = min(row, t);
                const uint32_t o = (uint32_t)row * ROWB + 16u * piece;
                kr[u] = *reinterpret_cast<const uint4*>(Ks + o);
                vr[u] = *reinterpret_cast<const uint4*>(Vs + o);
                blk += step_blk;
                in_blk += step_row;
                if (in_blk >= B) { in_blk -= B; ++blk; }
            }
        } else {
#pragma unroll
            for (int u = 0; u < NB; ++u) {
                const int pc = min(p0 + u * (NW * RPI) + kslot, total - 1), e = pc / B;
                const int64_t key = (int64_t)sel[e] * B + (pc - e * B);
                kr[u] = *reinterpret_cast<const uint4*>(Ks + key * ROWB + 16u * piece);
                vr[u] = *reinterpret_cast<const uint4*>(Vs + key * ROWB + 16u * piece);
            }
        }
        float z[NB], top = m;
#pragma unroll
        for (int u = 0; u < NB; ++u) {
            float a = 0.f;
            if constexpr (sizeof(T) == 2) {                 // (products exact, fp32 sums)
                const uint32_t w[4] = {kr[u].x, kr[u].y, kr[u].z, kr[u].w};
#pragma unroll
                for (int i = 0; i < 4; ++i) a = dot2(w[i], qb[i], a);
            } else {
                float f[EPL];
                widen(kr[u], f);
#pragma unroll
                for (int e = 0; e < EPL; ++e) a = fmaf(f[e], __uint_as_float(qb[e]), a);
            }
            z[u] = row_sum<LPR>(a) * c2;
            if (!ALL && p0 + u * (NW * RPI) + kslot >= total) {
                z[u] = -INFINITY;
                if (ZERO) vr[u] = make_uint4(0u, 0u, 0u, 0u);
            }
            top = fmaxf(top, z[u]);
        }
        // (a lane group without a key so far that exists and has a finite logit keeps m = -inf, l = 0: exponents
        // are taken against the lowest number, which leaves them -inf)
        const float ref = fmaxf(top, -3.402823466e+38f);
        const float alpha = __builtin_amdgcn_exp2f(m - ref);
        m = top;
        l *= alpha;
#pragma unroll
        for (int e = 0; e < EPL; ++e) acc[e] *= alpha;
#pragma unroll
        for (int u = 0; u < NB; ++u) {
            const float p = __builtin_amdgcn_exp2f(z[u] - ref);
            float f[EPL];
            widen(vr[u], f);
            l += p;
#pragma unroll
            for (int e = 0; e < EPL; ++e) acc[e] = fmaf(p, f[e], acc[e]);
        }
    };
    // Batches of eight instructions; the last few go into a batch of four where that holds them (rows past the end are
    // read like others).  Batches of ten for the ninth and tenth, of two, and a second batch on its way while one is
    // worked on were no better over the range of sizes.
    {
        constexpr int STEP = NW * RPI;
        using std::integral_constant;
        int p0 = first + wave * RPI;
        for (; p0 + 7 * STEP + RPI <= total; p0 += 8 * STEP) batch(p0, integral_constant<int, 8>(), std::true_type(), std::false_type());
        const int left = (total - p0 + STEP - 1) / STEP;             // instructions
        if (left > 4) batch(p0, integral_constant<int, 8>(), std::false_type(), std::false_type());
        else if (left > 0) batch(p0, integral_constant<int, 4>(), std::false_type(), std::false_type());
        // Weight 0 times an infinite value past the end is NaN.  A wave with a NaN does its keys once more, those values as zero, and
        // with the same results otherwise; clearing them in every last batch took 0.1 to 0.4 us of 15.
        float sum = acc[0];
#pragma unroll
        for (int e = 1; e < EPL; ++e) sum += acc[e];
        if (__ballot(sum != sum)) {
            m = -INFINITY;
            l = 0.f;
#pragma unroll
            for (int e = 0; e < EPL; ++e) acc[e] = 0.f;
            p0 = first + wave * RPI;
            blk = p0 / B;
            in_blk = p0 % B;
            for (; p0 < total; p0 += 8 * STEP) batch(p0, integral_constant<int, 8>(), std::false_type(), std::true_type());
        }
    }
    // ---- merge: the lane groups of a wave, then the waves through LDS
    auto weight = [](float a, float b) { return a == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(a - b); };
    auto add = [](float a, float b) { return a + b; };
    {
        const float top = across_rows<LPR>(m, [](float a, float b) { return fmaxf(a, b); });
        const float wt = weight(m, top);
        m = top;
        l = across_rows<LPR>(l * wt, add);
#pragma unroll
        for (int e = 0; e < EPL; ++e) acc[e] = across_rows<LPR>(acc[e] * wt, add);
    }
    float* mw = mrg + wave * (D + 2);
    if (lane == 0) { mw[0] = m; mw[1] = l; }
    if (kslot == 0) {
#pragma unroll
        for (int e = 0; e < EPL; ++e) mw[2 + piece * EPL + e] = acc[e];
    }
    __syncthreads();
    float top = -INFINITY, L = 0.f, o = 0.f;
    if (tid < D) {
#pragma unroll
        for (int w = 0; w < NW; ++w) top = fmaxf(top, mrg[w * (D + 2)]);
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const float wt = weight(mrg[w * (D + 2)], top);
            L = fmaf(wt, mrg[w * (D + 2) + 1], L);
            o = fmaf(wt, mrg[w * (D + 2) + 2 + tid], o);
        }
    }
    // ---- shares: the workgroup that is done last merges them, in their order
    if constexpr (SHARED) {
        // Everything shared goes through memory operations of agent scope, which other compute units see in whatever cache
        // they sit; the counter moves when the stores are through.  (A fence of agent scope would write back and drop
        // the whole L2: 20 -> 99 us with 64 queries shared by four workgroups each.)
        float* mine = split.part + (qrow * splits + share) * (D + 2);
        auto put = [](float* p, float x) { __hip_atomic_store(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
        if (tid < D) put(mine + 2 + tid, o);
        if (tid == 0) { put(mine, top); put(mine + 1, L); }
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(0);
        asm volatile("" ::: "memory");
        __syncthreads();
        if (tid == 0) {
            // A counter belongs to this launch if it carries its tag; anything else, whatever the memory held, is a
            // count of zero.  The last one leaves zero: a launch that is replayed carries the same tag again.
            uint64_t* at = split.arrived + qrow;
            uint64_t old = __hip_atomic_load(at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT), next;
            int before;
            do {
                before = (old >> 8) == split.tag ? (int)(old & 255u) : 0;
                next = before + 1 == splits ? 0u : split.tag << 8 | (uint64_t)(before + 1);
            } while (!__hip_atomic_compare_exchange_strong(at, &old, next, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                           __HIP_MEMORY_SCOPE_AGENT));
            ctl[0] = before + 1 == splits;
        }
        __syncthreads();
        if (!ctl[0]) return;
        if (tid < D) {
            float* theirs = split.part + qrow * splits * (D + 2);
            auto get = [](float* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
            float mx[kDecodeSplits], lx[kDecodeSplits], ox[kDecodeSplits];
#pragma unroll
            for (int x = 0; x < kDecodeSplits; ++x) {       // (all on their way at once)
                float* p = theirs + min(x, splits - 1) * (D + 2);
                mx[x] = get(p);
                lx[x] = get(p + 1);
                ox[x] = get(p + 2 + tid);
            }
            top = mx[0];
#pragma unroll
            for (int x = 1; x < kDecodeSplits; ++x) top = fmaxf(top, mx[x]);
            L = o = 0.f;
#pragma unroll
            for (int x = 0; x < kDecodeSplits; ++x) {       // (left out, not weighted by zero: a part may be infinite)
                if (x >= splits) break;
                const float wt = weight(mx[x], top);
                L = fmaf(wt, lx[x], L);
                o = fmaf(wt, ox[x], o);
            }
        }
    }
    if (tid < D) {
        O[qrow * D + tid] = from_f32<T>(o / L);
        if (tid == 0) lse[qrow] = (top + __builtin_amdgcn_logf(L)) * 0.6931471805599453f;
    }
}

// Workgroups per query.  A compute unit takes in a query's keys and values at about 25 bytes per clock whatever else is
// idle, so where there are few queries with much to read several units share one.  Each of them scores and selects for
// itself, which costs the others bandwidth: at most half the chip, and shares of 128 KB (up to 32 workgroups) or 256 KB.
// Whole call, us, unshared -> 2 / 4 / 8 workgroups per query: 4 queries of 1 MB 17.8 -> - / 15.9 / 14.4; 4 of 0.5 MB 15.7 ->
// 13.4 / 12.4 / 13.5; 16 of 1 MB 32.4 -> - / 26.8 / 28.3; 32 of 1.3 MB 40.4 -> - / 33.8 / 38.7; 64 of 0.9 MB 20.7 -> 17.9 / 18.8;
// 16 of 0.5 MB 14.3 -> 13.7 / 14.2; 64 of 0.5 MB 15.9 -> 15.8 / 17.3; 128 of 1 MB 30.3 -> 31.5; 32 of 0.27 MB 10.4 -> 12.8 (4).
// (The own block counts with the keys it has: 8 queries of 50 keys, in a block of 4096, take 8.1 us shared and 5.4 not.)
static int decode_splits(const Dims& s, int q_len)
{
    const int64_t queries = (int64_t)s.bh * q_len;
    const int64_t keys = (int64_t)std::min(s.k, (s.N - 1) / s.B) * s.B + (s.N - 1) % s.B + 1;     // of the last position
    const int64_t kb = 2 * keys * s.D * (s.dtype == MOBA_BF16 ? 2 : 4) >> 10;
    if (kb < 512) return 1;
    int n = 1;
    while (2 * n <= kDecodeSplits && 2 * n * queries <= 128 && kb >= 2 * n * (2 * n * queries <= 32 ? 128 : 256)) n *= 2;
    return n;
}
// [counters: one per query][partials: m, l, O of every share]
static size_t decode_counters_bytes(const Dims& s, int q_len) { return ((size_t)s.bh * q_len * sizeof(uint64_t) + 255) & ~(size_t)255; }
size_t decode_ws_bytes(const Dims& s, int q_len)
{
    const int n = decode_splits(s, q_len);
    return n == 1 ? 0 : decode_counters_bytes(s, q_len) + (size_t)s.bh * q_len * n * (s.D + 2) * sizeof(float);
}
// A number that launches hardly ever share (55 bits of a count, mixed).  Two that do are told apart all the same where the first is over,
// as it leaves zeros behind.
static uint64_t launch_tag()
{
    static std::atomic<uint64_t> launches{(uint64_t)std::chrono::steady_clock::now().time_since_epoch().count()};
    uint64_t x = launches.fetch_add(1, std::memory_order_relaxed) * 0x9e3779b97f4a7c15ull;
    x ^= x >> 32;
    return (x >> 8) | 1u;
}

template <typename T, int D>
static hipError_t decode_t(const Dims& s, int q_len, const void* Q, const void* K, const void* V,
                           const float* cent, int cblocks, void* O, float* lse, int32_t* idx, void* ws,
                           hipStream_t st)
{
    const int splits = ws ? decode_splits(s, q_len) : 1;
    DecodeSplit split = {nullptr, nullptr, 0};
    if (splits > 1) {
        split.arrived = static_cast<uint64_t*>(ws);
        split.part = reinterpret_cast<float*>(static_cast<char*>(ws) + decode_counters_bytes(s, q_len));
        split.tag = launch_tag();
    }
    const int npast_max = (s.N - 1) / s.B;
    const size_t lds = sizeof(float) * (size_t)((npast_max + 3) / 4 * 4 + kDecodeBins + kDecodeScratch<D> +
                                                (npast_max + 31) / 32 + 3 * kDecodeWaves + 5 + kDecodeGroups + s.k + 1);
    auto go = [&](auto* kernel) {
        if (lds > 64 * 1024) {
            const hipError_t e = ensure_dynamic_lds((const void*)kernel, lds);
            if (e != hipSuccess) return e;
        }
        hipLaunchKernelGGL(kernel, dim3((unsigned)schedule_grid(s.bhk, s.G * q_len * splits)), dim3(kDecodeThreads), lds, st,
                           (const T*)Q, (const T*)K, (const T*)V, cent, (T*)O, lse, idx, s.N, s.B, s.k, q_len,
                           cblocks, s.scale, s.G, s.bhk, npast_max, splits, split);
        return hipGetLastError();
    };
    if (s.k <= kDecodeShort) return splits > 1 ? go(decode_kernel<T, D, true, true>) : go(decode_kernel<T, D, false, true>);
    return splits > 1 ? go(decode_kernel<T, D, true, false>) : go(decode_kernel<T, D, false, false>);
}

hipError_t launch_decode(const Dims& s, int q_len, const void* Q, const void* K, const void* V,
                         const float* cent, int cblocks, void* O, float* lse, int32_t* idx, void* ws, hipStream_t st)
{
    if (s.dtype == MOBA_BF16)
        return s.D == 64 ? decode_t<bf16_t, 64>(s, q_len, Q, K, V, cent, cblocks, O, lse, idx, ws, st)
                         : decode_t<bf16_t, 128>(s, q_len, Q, K, V, cent, cblocks, O, lse, idx, ws, st);
    return s.D == 64 ? decode_t<float, 64>(s, q_len, Q, K, V, cent, cblocks, O, lse, idx, ws, st)
                     : decode_t<float, 128>(s, q_len, Q, K, V, cent, cblocks, O, lse, idx, ws, st);
}

}  // namespace moba
