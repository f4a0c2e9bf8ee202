// bf16 MFMA helpers for gfx950 (v_mfma_f32_16x16x32_bf16) and the operand layouts the
// attention kernels share.
//
// One MFMA multiplies A (16 x 32) by B (32 x 16) into C (16 x 16), fp32 accumulate.
// With lane = 16*g + m (g = 0..3, m = 0..15):
//   A operand: lane holds row m,  contraction slots 8g .. 8g+7   (8 bf16 = 4 VGPRs)
//   B operand: lane holds col m,  contraction slots 8g .. 8g+7
//   C result : lane holds col m,  rows 4g .. 4g+3                (4 fp32)
//
// Keys are processed in groups of 32 consecutive keys.  Scores are computed transposed,
// S^T = K_group (32 keys x d) . Q^T (d x 16 queries), as two 16-key tiles; a lane then
// holds, for its query column, keys {4g+i} of tile 0 and {16+4g+i} of tile 1.  Packed to
// bf16 in that order these 8 values ARE a B operand whose contraction slot s of group g
// means key  slot_key(g, s)  -- so the other operand of the next product only has to use
// the same slot order, and P never moves between lanes.
#pragma once
#include <type_traits>
#include <utility>

#include "common.h"

namespace moba {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

union Frag {               // one A or B operand
    bf16x8_t v;
    uint4 q;
    u32x4_t n;             // the same four registers as one native vector (asm operands)
    uint32_t u[4];
};

__device__ __forceinline__ f32x4_t mfma16(const Frag& a, const Frag& b, f32x4_t c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.v, b.v, c, 0, 0, 0);
}

// The 32 x 32 x 16 form.  With lane = 32*h + m:
//   A operand: lane holds row m, contraction slots 8h .. 8h+7 (B: col m)
//   C result : lane holds col m, element i is row 8 (i >> 2) + 4 h + (i & 3)
typedef float f32x16_t __attribute__((ext_vector_type(16)));
__device__ __forceinline__ f32x16_t mfma32(const Frag& a, const Frag& b, f32x16_t c)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.v, b.v, c, 0, 0, 0);
}

// LDS transpose read: within each group of 16 lanes, lane i receives as element e the 16-bit
// element (i & 3) of the 8 bytes that lane 4 e + (i >> 2) of the group points at.
__device__ __forceinline__ uint2 lds_read_tr16(const unsigned char* p)
{
    typedef short v4s __attribute__((ext_vector_type(4)));
    const v4s r = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        (__attribute__((address_space(3))) v4s*)(const_cast<unsigned char*>(p)));
    return *reinterpret_cast<const uint2*>(&r);
}

// key (0..31, inside its 32-key group) that contraction slot s of lane group g stands for
__host__ __device__ __forceinline__ constexpr int slot_key(int g, int s)
{
    return s < 4 ? 4 * g + s : 16 + 4 * g + (s - 4);
}

// channel that row m of M-tile mt of a (d x 16) product stands for: the four lane groups of such a
// result (rows 4g'..4g'+3) hold D/4 consecutive channels each.
template <int D>
__host__ __device__ __forceinline__ constexpr int tile_chan(int mt, int m)
{
    return (m >> 2) * (D / 4) + 4 * mt + (m & 3);
}

// word 16 mt + m of a query tile's accumulator row (channel tile_chan(mt, m)) that holds channel c
template <int D>
__host__ __device__ __forceinline__ constexpr int acc_word(int c)
{
    return 16 * (c % (D / 4) / 4) + 4 * (c / (D / 4)) + (c & 3);
}

__device__ __forceinline__ uint32_t pack2(float lo, float hi)
{
    // round to nearest even, two at a time
    return pack_bf16x2(lo, hi);
}

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ float fast_log2(float x) { return __builtin_amdgcn_logf(x); }

// exponent e with |x| * 2^-e <= 1 for every |x| <= vmax (vmax >= 0 given as fp32 bits)
__device__ __forceinline__ int scale_exponent(uint32_t vmax_bits)
{
    const int E = (int)((vmax_bits >> 23) & 0xffu);
    return E == 0 ? 0 : E - 127 + 1;
}

// maximum that hands a NaN on (v_maximum3_f32 on gfx950; fmaxf would drop it)
__device__ __forceinline__ float max_nan(float a, float b) { return __builtin_elementwise_maximum(a, b); }
// the value of lane FROM of this lane's group of GROUP (a power of two up to 32) neighbouring lanes
template <int GROUP, int FROM>
__device__ __forceinline__ float from_lane_of_group(float x)
{
    return __int_as_float(__builtin_amdgcn_ds_swizzle(__float_as_int(x), FROM << 5 | (31 & ~(GROUP - 1))));
}
// sum and maximum (NaN-propagating) of a lane's value and that of the lane 32 away
__device__ __forceinline__ float sum_halves(float x)
{
    const uint32_t b = __float_as_uint(x);
    const auto r = __builtin_amdgcn_permlane32_swap(b, b, false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float max_halves(float x)
{
    const uint32_t b = __float_as_uint(x);
    const auto r = __builtin_amdgcn_permlane32_swap(b, b, false, false);
    return max_nan(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
// channel maximum (fp32 bits of a magnitude) of a tensor that holds an infinity or a NaN
__device__ __forceinline__ bool nonfinite_bits(uint32_t magnitude_bits) { return magnitude_bits >= 0x7f800000u; }

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

// Element offset of the "slot-ordered transposed" copy of a [N, D] tensor X (keys or values):
// for 32-row group kap, M-tile mt, lane (g, m), slot s it holds X[32*kap + slot_key(g,s)][tile_chan(mt,m)],
// stored so that the 64 lanes of one (kap, mt) read 1 KB contiguously, 16 B per lane.
template <int D>
__host__ __device__ __forceinline__ constexpr int64_t slot_major_offset(int64_t kap, int mt, int lane)
{
    return (kap * (D / 16) + mt) * 512 + (int64_t)lane * 8;
}

// An entry of a tile's offs[]: where the block's rows start in rows8 (a multiple of 4, so that four
// of them are one aligned word) and how many there are.
__device__ __forceinline__ int list_start(uint32_t o) { return (int)(o & 0xffffu); }
__device__ __forceinline__ int list_count(uint32_t o) { return (int)(o >> 16); }

// Ascending list of the non-empty blocks of a set of row lists (offs as built below):
// ulist[0 .. *count).  All NT threads; ends with a workgroup barrier.
template <int NT>
__device__ __forceinline__ void list_nonempty(const uint32_t* offs, int nb, uint16_t* ulist,
                                              int* count, uint32_t* wsum, int tid)
{
    const int lane = tid % kWave, wave = tid / kWave;
    int base = 0;
    for (int c = 0; c < nb; c += NT) {
        const int i = c + tid;
        const bool some = i < nb && list_count(offs[i]) > 0;
        const uint64_t b = __ballot(some);
        if (lane == 0) wsum[wave] = (uint32_t)__popcll(b);
        __syncthreads();
        int before = 0, total = 0;
#pragma unroll
        for (int wv = 0; wv < NT / kWave; ++wv) {
            const int n = (int)wsum[wv];
            if (wv < wave) before += n;
            total += n;
        }
        if (some) ulist[base + before + lanes_below(b)] = (uint16_t)i;
        base += total;
        __syncthreads();
    }
    if (tid == 0) *count = base;
    __syncthreads();
}

// Next entry of a work list shared by the waves of a workgroup (the same value in all lanes).
// Units differ in length and the memory system does not serve all waves alike, so a static
// deal leaves waves idle at the barrier that ends the list.
__device__ __forceinline__ int take_unit(int* counter, int lane)
{
    int e = 0;
    if (lane == 0) e = atomicAdd(counter, 1);
    return __builtin_amdgcn_readfirstlane(e);
}

// ---- per-tile block lists in LDS --------------------------------------------------------
// For a tile of TILE consecutive queries and the key blocks [lo, hi): a counting sort of the
// tile's (row, kept block) pairs by block.  Afterwards offs[j - lo] says which piece of rows8[]
// holds the local rows (0 .. TILE-1, one byte each) that kept block j, in no
// particular order.  Built once per tile and range, by all NT threads; integer atomics only.
//   cur   [hi - lo + 1] words of scratch (counters, then insertion cursors)
//   offs  [hi - lo] words
//   rows8 cap < 65536 bytes; a routing without repeats has at most min(TILE * (hi - lo), TILE * k)
//         pairs, a block's list takes up to three bytes more, and pairs beyond cap are dropped
//         rather than written
//   wsum  NT / 64 words of scratch
// `idx_tile` points at the tile's first topk_idx row; entries that are not past blocks of
// their row are ignored.  Ends with a workgroup barrier.
template <int TILE, int NT>
__device__ __forceinline__ void build_block_lists(const int32_t* __restrict__ idx_tile, int t0,
                                                  int rows_here, int k, int B, int lo, int hi,
                                                  uint32_t* cur, uint32_t* offs, uint8_t* rows8,
                                                  uint32_t cap, uint32_t* wsum, int tid)
{
    constexpr int TPR = NT / TILE;                 // threads per row
    const int nb = hi - lo;
    const int r = tid / TPR, part = tid % TPR;
    const int past = (t0 + r) / B;
    const int lane = tid % kWave, wave = tid / kWave;
    auto for_each_entry = [&](auto f) {
        if (r >= rows_here) return;
        const int32_t* row = idx_tile + (int64_t)r * k;
        auto one = [&](int b) { if (b >= lo && b < hi && b < past) f(b - lo); };
        if ((k & 3) == 0) {                        // 16-byte loads, several in flight
            const int4* row4 = reinterpret_cast<const int4*>(row);
            const int n4 = k >> 2;
            for (int e0 = part; e0 < n4; e0 += 4 * TPR) {
                int4 v[4];
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    v[j] = e0 + j * TPR < n4 ? row4[e0 + j * TPR] : make_int4(-1, -1, -1, -1);
#pragma unroll
                for (int j = 0; j < 4; ++j) { one(v[j].x); one(v[j].y); one(v[j].z); one(v[j].w); }
            }
        } else {
            for (int e = part; e < k; e += TPR) one(row[e]);
        }
    };
    for (int i = tid; i <= nb; i += NT) cur[i] = 0u;
    __syncthreads();
    for_each_entry([&](int j) { atomicAdd(&cur[j], 1u); });
    __syncthreads();
    // exclusive scan of the counts: each thread takes EPT consecutive blocks
    constexpr int kMaxRange = 1024;
    constexpr int EPT = (kMaxRange + NT - 1) / NT;
    uint32_t v[EPT], sum = 0;
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
        const int j = tid * EPT + e;
        v[e] = j < nb ? cur[j] : 0u;
        sum += (v[e] + 3u) & ~3u;
    }
    uint32_t incl = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t t = __shfl_up(incl, o, 64);
        if (lane >= o) incl += t;
    }
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    uint32_t base = incl - sum;
    for (int wv = 0; wv < wave; ++wv) base += wsum[wv];
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
        const int j = tid * EPT + e;
        if (j < nb) {
            const uint32_t start = min(base, cap);
            offs[j] = start | (min(v[e], cap - start) << 16);
            cur[j] = base;
        }
        base += (v[e] + 3u) & ~3u;
    }
    __syncthreads();
    for_each_entry([&](int j) {
        const uint32_t pos = atomicAdd(&cur[j], 1u);
        if (pos < cap) rows8[pos] = (uint8_t)r;
    });
    __syncthreads();
}

// Sixteen listed rows as the columns (or rows) of a product: column m takes the row at place listed_at(m) of the
// sixteen.  The product's result rows 4 g + i, i fixed, are then the places 4 i + g: instruction i of the adds covers
// four neighbouring places, and a list's last sixteen needs no more of these instructions than it has rows / 4: 5.8 -> 4.4 of them
// per channel tile and list of about sixteen rows.  Long lists only pay for it: taken where lists have up to `line` rows
// on average, by the shape (d = 64; d = 128, dense, 3 heads of 2176: dQ 155 -> 163 us).
// us without -> with it, at so many rows a list: forward (B = 32) 16 201.5 -> 197.3; 31 966.7 -> 947.0; 38 97.9 -> 97.6;
// 66 225.8 -> 228.6; 87 159.7 -> 160.3; 254 206.5 -> 212.5.  dQ 20 760.5 -> 754.7; 31 910.0 -> 882.4; 60 (hot blocks) 783.4 -> 771.5;
// 87 151.2 -> 148.9 (B = 64: 152.8 -> 152.3); 148 160.5 -> 158.0 (B = 128: 248.8 -> 251.5, B = 256: 103.5 -> 105.3); 254 155.9 -> 159.9.
constexpr int kShortListsForward = 48, kShortListsDq = 128;
inline bool short_lists(const Dims& s, int tile, int line)
{
    const int64_t tiles = (s.N + tile - 1) / tile;
    return 2 * s.R <= line * tiles * s.n;                   // half of all (tile, block) pairs are past blocks
}
__device__ __forceinline__ int listed_at(int m) { return 4 * (m & 3) + (m >> 2); }
// the rows at places 4 i + g, i = 0 .. 3, from what the lane (g, m16) read at place 4 (m16 & 3) + g
__device__ __forceinline__ void listed_rows(int at, int (&r4)[4])
{
    r4[0] = __builtin_amdgcn_mov_dpp(at, 0x00, 0xf, 0xf, true);         // quad_perm: lane i of every four
    r4[1] = __builtin_amdgcn_mov_dpp(at, 0x55, 0xf, 0xf, true);
    r4[2] = __builtin_amdgcn_mov_dpp(at, 0xaa, 0xf, 0xf, true);
    r4[3] = __builtin_amdgcn_mov_dpp(at, 0xff, 0xf, 0xf, true);
}

// f(integral_constant 0), f(integral_constant 1), ...
template <typename F, int... I>
__device__ __forceinline__ void unrolled(std::integer_sequence<int, I...>, F f)
{
    (f(std::integral_constant<int, I>{}), ...);
}

// ---- merging a query's partials (attn_fwd_km.hip, attn_bwd_km.hip) ---------------------------
// D / 8 neighbouring lanes share a query; its partials [e][c] lie side by side and are taken CH at a time,
// every load unconditional (past the end: the last one again, ignored), so that a lane has CH
// 16-byte loads in flight.  What goes with a partial -- is it there, its (m, l) -- is looked up once per
// query, by the lane that stands at its place in the chunk.  (Every lane looking up every partial for itself
// kept the address and data units busy all the time: 4.4 of 4.4 ms at 151 M partials of d = 64.)
// The partials are streamed: nothing reads them again.  Part of what that saves comes back in the next kernel, which
// finds the memory system still busy; the sum is the smaller one.  us, plain -> streaming loads, 32 slices, d = 64,
// B = 128, k = 8: N = 65536 forward merge 580 -> 565, row sums D after it 101 -> 115; dQ merge 534 -> 492, centroids of the
// next step after it 53 -> 78; N = 524288 4467 -> 4345, 790 -> 801; 4148 -> 3927, 372 -> 406; N = 16384 167 -> 127, 27 -> 25;
// 142 -> 113, 16 -> 13.  Steps: 5.56 -> 5.52, 56.9 -> 56.7, 1.35 -> 1.29 ms.
template <int D>
struct MergeRow {
    static constexpr int LANES = D / 8, ROWS = 256 / LANES;             // a query's lanes; queries of a workgroup
    int64_t row;                                                        // slice * N + t
    int lane, piece, own_parts, slots, k, nsub;
    const int32_t* irow;

    // ROWS divides B and with it N: a workgroup's queries lie in one slice
    __device__ __forceinline__ MergeRow(const int32_t* idx, int N, int B, int k_, int nsub_, int part_keys)
        : lane(threadIdx.x % kWave), piece(threadIdx.x % LANES), slots((k_ + 1) * nsub_), k(k_), nsub(nsub_)
    {
        row = (int64_t)blockIdx.x * ROWS + threadIdx.x / LANES;
        own_parts = 1;
        if (nsub > 1) {
            const int t = (int)(blockIdx.x % (uint32_t)(N / ROWS)) * ROWS + (int)(threadIdx.x / LANES);
            own_parts = (t % B) / part_keys + 1;
        }
        irow = idx + row * k;                                            // (k = 0: never read)
    }
    // is slot si there?  Its block was kept; of the own block: the parts up to the query's own key
    __device__ __forceinline__ bool counts(int si) const
    {
        int e = si, c = 0;
        if (nsub > 1) { e = si / nsub; c = si - e * nsub; }
        const int j = k > 0 ? irow[min(e, k - 1)] : 0;
        return si < slots && (e == k ? c < own_parts : j >= 0);
    }
};
// Partials per chunk, one of the instantiated sizes: the one with the fewest loads past a query's end, the larger of two
// that are equal.  Merge alone, 8 slices of N = 16384, B = 64, us with 4 / 6 / 9 / 11 / 13, forward | dQ:
//   d = 64,  5 partials  21.8 17.9 22.0 29.8 26.4 | 19.7 18.5 21.2 23.9 25.5    9  35.7 32.9 32.5 34.5 34.4 | 31.9 31.1 28.3 29.3 31.2
//           11  35.4 33.2 43.9 38.0 37.4 | 34.0 33.5 39.6 34.3 32.9            17  61.7 53.6 58.1 63.5 67.3 | 52.7 50.0 50.6 53.0 57.3
//           33  116 111 117 105 114 | 112 110 110 106 110                      65  233 221 244 218 215 | 218 215 219 214 212
//   d = 128, 9  68.0 58.3 59.9 64.7 59.5 | 59.6 56.4 55.7 55.2 59.6           17  115 105 110 121 119 | 110 108 107 109 115
//           33  194 208 204 198 210 | 210 209 206 205 208                      65  373 379 382 383 385 | 406 403 393 402 395
// Of 41 counts the pick is within 3 % of the best size in 39 (dQ) and 27 (forward: chunks of 9 and 11 at d = 64 are up to
// 8 % behind those of 6 at 17 and 18 partials and 14 % at 10 and 11, and ahead of them from 33 partials on; runs of
// this table, which has the launch in it, differ by 2 to 3 %).
inline int merge_chunk(int slots)
{
    int best = 13;
    for (int c : {11, 9, 6, 4})
        if ((slots + c - 1) / c * c < (slots + best - 1) / best * best) best = c;
    return best;
}

// ---- prepared copies of K and V (prepare.hip) ------------------------------------------------
// "MFMA operand order": the 16 bytes lane (m, g) feeds to the MFMA as rows 16 mt + m, channels
// 32 ks + 8 g .. + 8 of 32-key group kap sit at ((kap * 2 + mt) * (D / 32) + ks) * 1024 + 16 * lane.
// One load instruction of a wave then covers 1 KB of consecutive bytes; reading the same operand
// from the row-major tensor (16 rows x 64 bytes per instruction) runs at a quarter of that rate on
// this chip.  "Slot-ordered transposed": slot_major_offset() above.
struct Prepared {
    uint32_t* kmax = nullptr;   // [bhk][D] largest magnitude per channel of K, fp32 bits
    uint32_t* vmax = nullptr;   //                                          of V
    void* Ka = nullptr;         // K in MFMA operand order
    void* Vt = nullptr;         // V slot-ordered transposed, scaled per channel
    void* Kt = nullptr;         // K slot-ordered transposed, scaled per channel
    void* Va = nullptr;         // V in MFMA operand order
};
constexpr unsigned kPrepKa = 1, kPrepVt = 2, kPrepKt = 4, kPrepVa = 8;
constexpr unsigned kPrepForward = kPrepKa | kPrepVt;             // what the query-tile forward reads
constexpr unsigned kPrepBackward = kPrepKa | kPrepKt | kPrepVa;  // what the query-tile dQ kernel reads
constexpr unsigned kPrepAll = kPrepForward | kPrepBackward;
size_t prepared_layout(const Dims& s, unsigned mask, void* base, Prepared* out);
// makes the parts of `p` that are not null (the maxima it needs first)
hipError_t launch_prepare(const Dims& kv, const void* K, const void* V, const Prepared& p, hipStream_t st);
bool shared_workspace(const Dims& s);

size_t forward_mfma_ws_bytes(const Dims& s);
hipError_t launch_forward_mfma(const Dims& s, const void* Q, const void* K, const void* V,
                               void* ws, const int32_t* idx, const int32_t* off, const int32_t* ql,
                               void* O, float* lse, hipStream_t st);

size_t backward_mfma_ws_bytes(const Dims& s);
hipError_t launch_dq_mfma(const Dims& s, const void* Q, const void* K, const void* V, const void* dO,
                          const float* lse, const int32_t* idx, const int32_t* off, const int32_t* ql,
                          void* dQ, void* ws, hipStream_t st);

// ld: per query (lse log2 e, -D), as the D kernel packs them; part: dkdv_heads_ws_bytes() of
// scratch for the per-query-head sums when key/value heads are shared (unused otherwise)
size_t dkdv_heads_ws_bytes(const Dims& s);
hipError_t launch_dkdv_mfma(const Dims& s, const void* Q, const void* K, const void* V,
                            const void* dO, const float2* ld, const int32_t* off,
                            const int32_t* ql, void* dK, void* dV, float* part, hipStream_t st);

hipError_t launch_dkdv_heads(const Dims& s, const float* part, void* dK, void* dV, hipStream_t st);

size_t topk_mfma_ws_bytes(const Dims& s);
bool topk_mfma_supported(const Dims& s);
hipError_t launch_topk_mfma(const Dims& s, const void* Q, const float* cent, int32_t* idx, void* ws,
                            hipStream_t st);

// gate for rows of at most 64 kept blocks (gate_mfma.hip); the terms it shares with topk_mfma.hip
bool gate_supported(const Dims& s);
size_t gate_ws_bytes(const Dims& s);
hipError_t launch_gate(const Dims& s, const void* Q, const float* cent, int32_t* idx, void* ws, hipStream_t st);
hipError_t launch_split3(const Dims& s, const float* cent, bf16_t* c3, float4* norms, int32_t* redo, hipStream_t st);
hipError_t launch_topk_redo(const Dims& s, const void* Q, const bf16_t* c3, const int32_t* redo, int32_t* idx,
                            hipStream_t st);

constexpr int kKeyMajorMaxTopk = 64;      // longest row of kept blocks the key-major kernels take

// keys a key-major workgroup holds in registers as MFMA operands: the whole block up to 128
// (d = 64) or 64 (d = 128) keys, else parts of that size
__host__ __device__ inline int km_part_keys(int B, int D)
{
    const int cap = D == 64 ? 128 : 64;
    return B <= cap ? B : cap;
}

// workspace parts start on 256-byte boundaries
inline size_t a256(size_t x) { return (x + 255) & ~(size_t)255; }

// (query, kept block or own block, part of the block) triples: the partial results of the
// key-major kernels, [bh][N][k+1][parts]
inline size_t km_partials(const Dims& s)
{
    return (size_t)s.bh * s.N * (size_t)(s.k + 1) * (size_t)(s.B / km_part_keys(s.B, s.D));
}

// shapes the MFMA kernels cover: bf16 I/O and key blocks made of whole 32-key groups
inline bool mfma_path(const Dims& s)
{
    return s.dtype == MOBA_BF16 && s.B % 32 == 0 && !(s.flags & MOBA_FLAG_REFERENCE_KERNELS);
}

// The query-tile forward accumulates the row sums and P V as 32-bit fixed point with
// F = 30 - bitlen(keys a query can attend) fraction bits, the 32 keys of a row and group per add
// (the channel sums of P V likewise): a partial sum below 2^-(F+1) is lost, so a row with one
// dominant logit beside very many tiny ones can lose up to keys * 2^-(F+6) of its denominator (the
// sum is biased: every term is positive).  With at most 4096 keys per query F is at least 17 and
// that loss at most 0.05 % in the worst case (16384 keys would allow 0.4 %, 32768 keys 1.6 %,
// which shows in the output); longer rows go to the key-major or the plain kernels, which keep
// their sums in floating point.
constexpr int64_t kTileForwardMaxKeys = 4096;
inline int64_t keys_per_query(const Dims& s)
{
    const int64_t kept = (int64_t)(s.k + 1) * s.B;
    return kept < s.N ? kept : s.N;
}
inline bool tile_forward_ok(const Dims& s) { return keys_per_query(s) <= kTileForwardMaxKeys; }

// shapes the key-major kernels cover: key blocks of one part or of whole parts
inline bool key_major_shape(const Dims& s)
{
    return mfma_path(s) && s.B % km_part_keys(s.B, s.D) == 0 && s.k <= kKeyMajorMaxTopk;
}

// Query-tile or key-major attention?  Both are priced per query from fits to measured times (ns
// per query and slice on the whole chip, forward and dQ averaged; a wrong pick near the line costs
// 10-20 %):
//   tiles      c0 + k (B / 32) (g0 + g1 / rows): a tile of T consecutive queries (256 for d = 64,
//              128 for d = 128) meets a past key block with rows = T k / n of its rows and pays
//              per 32-key group at least a 16-row MFMA tile and the group's operands;
//   key-major  c (k + 1) (1 + 0.7 (parts - 1)): the gathered row, the partial result written and
//              read back per (query, block) pair, whatever B, and again for every further part of
//              the block.
// With k = 8 of B = 128 key-major wins from N = 8K on; with k = 64 of B = 32 (many blocks per
// query, every pair a partial in memory) the tiles win up to N of a few hundred thousand.
inline bool key_major_path(const Dims& s)
{
    if (!key_major_shape(s) || (s.flags & MOBA_FLAG_QUERY_TILES)) return false;
    if (s.flags & MOBA_FLAG_KEY_MAJOR) return true;
    if (!tile_forward_ok(s)) return true;
    if (s.k <= 0) return false;
    const bool d64 = s.D == 64;
    const double T = d64 ? 256.0 : 128.0;
    const double rows = T * s.k * (double)s.B / (double)s.N;
    const double parts = (double)(s.B / km_part_keys(s.B, s.D));
    const double tiles = (d64 ? 0.6 : 1.1) + 0.0013 * s.B +
                         s.k * (s.B / 32.0) * (d64 ? 0.015 + 0.14 / rows : 0.033 + 0.272 / rows);
    const double keymajor = (d64 ? 0.115 : 0.17) * (s.k + 1) * (1.0 + 0.7 * (parts - 1.0));
    return keymajor < tiles;
}

// The caller gives forward and backward the same workspace and the forward call prepares for both:
// only where both run on the query-tile kernels.
inline bool shared_workspace(const Dims& s)
{
    return (s.flags & MOBA_FLAG_SHARED_WORKSPACE) && mfma_path(s) && tile_forward_ok(s) && !key_major_path(s);
}

// Key-block-major attention on fp32 matrix cores (attn_f32_km.hip): fp32 tensors, and bf16 ones outside
// mfma_path()
bool f32_km_path(const Dims& s);
size_t forward_f32_km_ws_bytes(const Dims& s);
size_t backward_f32_km_ws_bytes(const Dims& s);
size_t backward_f32_km_ld_offset(const Dims& s);
hipError_t launch_forward_f32_km(const Dims& s, const void* Q, const void* K, const void* V, void* ws,
                                 const int32_t* idx, const int32_t* off, const int32_t* ql, void* O, float* lse,
                                 hipStream_t st);
hipError_t launch_backward_f32_km(const Dims& s, const void* Q, const void* K, const void* V, const void* dO,
                                  const int32_t* idx, const int32_t* off, const int32_t* ql, void* dQ, void* dK,
                                  void* dV, void* ws, uint32_t parts, hipStream_t st);
// shapes whose kernels file results by (query, place of the block in its row): the lists carry the place
inline bool lists_with_places(const Dims& s) { return key_major_path(s) || f32_km_path(s); }

size_t forward_km_ws_bytes(const Dims& s);
size_t backward_km_ws_bytes(const Dims& s);
hipError_t launch_backward_km(const Dims& s, const void* Q, const void* K, const void* V, const void* dO,
                              const float2* ld, const int32_t* idx, const int32_t* off, const int32_t* ql, void* dQ,
                              void* dK, void* dV, float* part, void* ws, hipStream_t st);
hipError_t launch_forward_km(const Dims& s, const void* Q, const void* K, const void* V, void* ws,
                             const int32_t* idx, const int32_t* off, const int32_t* ql, void* O,
                             float* lse, hipStream_t st);

}  // namespace moba
