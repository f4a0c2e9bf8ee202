// MoBA attention on fp32 matrix cores, key-block major, forward and backward: for fp32 tensors, and
// for bf16 tensors whose key blocks are not whole 32-key groups (the bf16 MFMA kernels' unit).  The
// cut is that of attn_fwd_km.hip: a workgroup owns up to 64 keys of one key block (paper Section 4.2:
// key blocks outermost, their routed queries gathered into dense tiles) and walks the block's query
// list, then the block's own queries under the causal mask, 16 queries per step and wave; a query's
// contributions from different key blocks are written once, as fp32 rows [query][kept block][part],
// and a merge kernel adds them up in a fixed order.  The place of a kept block comes with the list entry, and
// is looked up in the query's row where the lists were built for other kernels and do not hold it.  v_mfma_f32_16x16x4_f32 everywhere: fp32 operands,
// products and sums.
//
// The plain kernels of attn_reference.hip, which served these shapes, read every key row again for
// every query (64 FMAs per 256 bytes) and ran at 5 TFLOP/s; here a key row meets 16 queries per read.
// What bounds them now is the latency between the dependent steps of few waves, and the longest walks: at the shape below the matrix
// pipe is busy 57 % (forward) and 66 % (backward) of the clocks, the LDS pipe 19 %, VALU issue 26 and 24 %, and waves wait 64 % of their
// cycles; the products of the backward alone would take 68 of its 123 us.
// fp32, 2 x 4 heads, N = 4096, d = 64, B = 64, k = 7: forward 580 -> 74 us, backward 1960 -> 147 us.
//
// Operand layouts (lane = 16 g + m): a contraction over channels takes channels 16 t + 4 g + i in the
// i-th of four instructions, so that one 16-byte read per lane feeds four; a contraction over keys (or
// queries) takes rows 4 g + i, which is where the result layout of the product before has them, and
// its other operand comes from a row-major tile with output channel 4 m + mt, one 16-byte read for the
// four instructions mt = 0 .. 3.  Tiles in LDS have rows of D + 4 words: both reads are conflict-free.
#include <algorithm>
#include <cmath>

#include "mfma.h"

namespace moba {

namespace {

__device__ __forceinline__ f32x4_t mfma4(float a, float b, f32x4_t c)
{
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

constexpr float kFltLargest = 3.402823466e+38f;

template <int D>
struct F32Cfg {
    static constexpr int LD = D + 4;                   // words per row of a tile in LDS
    static constexpr int MT = D / 16;                  // 16-channel tiles of a row
    static constexpr int H = D / 64;                   // 16-byte reads per lane and transposed row
    static constexpr int NWF = 4;                      // waves per workgroup, forward
    static constexpr int NWB = D == 64 ? 8 : 4;        // backward
    static constexpr size_t fwd_lds(int nt) { return sizeof(float) * LD * (size_t)(2 * 16 * nt + NWF * 16); }
    static constexpr int bwd_wave_words(int nt) { return 2 * 16 * LD + 16 * (16 * nt + 4) + 32; }
    static constexpr size_t bwd_lds(int nt)
    {
        return sizeof(float) * ((size_t)2 * 16 * nt * LD + (size_t)NWB * bwd_wave_words(nt));
    }
};

// how a row of T comes in: CPR lanes of 16 bytes, RPI rows per load instruction, NI instructions for 16 rows
template <typename T, int D>
struct Gather {
    static constexpr int CPR = D * (int)sizeof(T) / 16, RPI = kWave / CPR, NI = 16 / RPI, EPL = 16 / (int)sizeof(T);
};

// the 16 bytes of a lane as fp32 to LDS
template <typename T>
__device__ __forceinline__ void put(float* dst, const u32x4_t& x)
{
    if constexpr (sizeof(T) == 4) {
        *reinterpret_cast<u32x4_t*>(dst) = x;
    } else {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            u32x4_t y;
            y[0] = x[2 * h] << 16; y[1] = x[2 * h] & 0xffff0000u;
            y[2] = x[2 * h + 1] << 16; y[3] = x[2 * h + 1] & 0xffff0000u;
            *reinterpret_cast<u32x4_t*>(dst + 4 * h) = y;
        }
    }
}

// the first ROWS rows of X -> tile[row][D + 4]; rows nk and beyond read as zero.  True: this thread
// brought an infinity or a NaN
template <typename T, int D, int ROWS, int NTHREADS>
__device__ __forceinline__ bool stage_rows(const T* __restrict__ X, float* tile, int nk, int tid)
{
    constexpr int CPR = Gather<T, D>::CPR, EPL = Gather<T, D>::EPL;
    uint32_t top = 0u;                                      // largest magnitude, as bits: infinities and NaN come last
    constexpr int IT = (ROWS * CPR + NTHREADS - 1) / NTHREADS;
    u32x4_t all[IT];                                        // (requested together: forward at d = 128 818 -> 758 us)
#pragma unroll
    for (int u = 0; u < IT; ++u) {
        const int i = tid + u * NTHREADS;
        all[u] = *reinterpret_cast<const u32x4_t*>(X + (size_t)min(i / CPR, nk - 1) * D + i % CPR * EPL);
    }
#pragma unroll
    for (int u = 0; u < IT; ++u) {
        const int i = tid + u * NTHREADS, r = i / CPR, c = i % CPR;
        if (ROWS * CPR % NTHREADS != 0 && r >= ROWS) break;
        const u32x4_t x = r < nk ? all[u] : u32x4_t{0u, 0u, 0u, 0u};
        put<T>(tile + r * (D + 4) + c * EPL, x);
#pragma unroll
        for (int h = 0; h < 4; ++h) {
            top = max(top, x[h] & 0x7fffffffu);
            if constexpr (sizeof(T) == 2) top = max(top, x[h] << 16 & 0x7fffffffu);
        }
    }
    return top >= 0x7f800000u;
}

// A key that a query does not see has weight zero, and the matrix instructions add 0 * x for it: no zero where x
// is an infinity or a NaN.  Only a block's own queries fail to see keys of it.  So where a part holds such a
// value, every wave does the own rows of its walk once more afterwards, one query at a time over the keys that
// it sees: f(query, number of keys of the part that it sees).
// It works out afresh where it is, from a block and thread number that the compiler cannot know to be the same:
// what it shares with the walk would be kept in registers all along that, 3 % of the forward at d = 128.
struct OwnRows {
    int s, c, lane, wave, a0, stride, nlist, total, own0, nk;
    int64_t q0, kv0;                                        // rows of the slice's first query, of the part's first key
    __device__ __forceinline__ OwnRows(const int32_t* __restrict__ off, int N, int B, int n, int nsub, int pk, int nsplit, int bh,
                                       int G, int waves)
    {
        int tid = threadIdx.x, block = blockIdx.x, u;
        asm volatile("" : "+v"(tid), "+s"(block));
        lane = tid % kWave;
        wave = tid / kWave;
        schedule(block, bh, n * nsub * nsplit, s, u);
        const int jc = u / nsplit, j = jc / nsub;
        c = jc - j * nsub;
        nk = min(pk, B - c * pk);
        own0 = j * B + c * pk;
        const int32_t* os = off + (int64_t)s * (n + 1) + j;
        nlist = os[1] - os[0];
        total = nlist + (B - c * pk);
        a0 = 16 * (u % nsplit * waves + wave);
        stride = 16 * waves * nsplit;
        q0 = (int64_t)s * N;
        kv0 = (int64_t)(s / G) * N + own0;
    }
    template <typename F>
    __device__ __forceinline__ void again(F f)
    {
        __threadfence_block();                              // (the walk's partials go first)
#pragma unroll 1
        for (; a0 < total; a0 += stride)
#pragma unroll 1
            for (int a = max(a0, nlist); a < min(a0 + 16, total); ++a) f(own0 + (a - nlist), min(a - nlist + 1, nk));
    }
};

template <typename T, int D>
__device__ __forceinline__ float row_dot(const T* __restrict__ a, const T* __restrict__ b)
{
    float acc = 0.f;
#pragma unroll 1
    for (int c = 0; c < D; c += 8) {
        float x[8], y[8];
        Vec8<T>::load(a + c, x);
        Vec8<T>::load(b + c, y);
#pragma unroll
        for (int e = 0; e < 8; ++e) acc = fmaf(x[e], y[e], acc);
    }
    return acc;
}

// out[0 .. D) <- the weights (a lane each, the first `seen` lanes) times as many rows of X; w: 64 words of LDS
template <typename T, int D>
__device__ __forceinline__ void weigh_rows(float weight, int seen, const T* __restrict__ X, float* w, float* out, int lane)
{
    w[lane] = weight;
    __builtin_amdgcn_wave_barrier();
#pragma unroll 1
    for (int ch = lane; ch < D; ch += kWave) {
        float acc = 0.f;
#pragma unroll 1
        for (int u = 0; u < seen; ++u) acc = fmaf(w[u], to_f32<T>(X[(size_t)u * D + ch]), acc);
        out[ch] = acc;
    }
    __builtin_amdgcn_wave_barrier();
}

// the walk of a workgroup: positions 0 .. nlist - 1 are the block's list, then its own queries from the
// part's first key on; positions past the end read as the first own query
struct Walk {
    const int32_t* src;
    int nlist, llast, own0, own_e, total;
    __device__ __forceinline__ int at(int a) const
    {
        const int listed = src[min(a, llast)];
        const int t = a < nlist ? listed : (own0 + (a - nlist)) | own_e;
        return a >= total ? own0 | own_e : t;
    }
};

// Where block j stands in the query's row of kept blocks (own rows: k).  The list entry says it where the
// lists were built for these kernels; lists built for others say 0.  `there` is what the row holds at the
// place of the entry; if that is not j, the row is searched.  -1: the row does not hold j.
__device__ __forceinline__ int place_of(int entry, int there, const int32_t* __restrict__ irow, int j, int k)
{
    int e = list_slot(entry);
    if (e >= k || there == j) return e;
    for (e = k - 1; e >= 0 && irow[e] != j; --e) {}
    return e;
}

}  // namespace

// NT: 16-key tiles of a part
template <typename T, int D, int NT>
__global__ __launch_bounds__(F32Cfg<D>::NWF * kWave) void fwd_f32_km_kernel(
    const T* __restrict__ Q, const T* __restrict__ K, const T* __restrict__ V, const int32_t* __restrict__ idx,
    const int32_t* __restrict__ off, const int32_t* __restrict__ ql, float* __restrict__ PO, float2* __restrict__ Pml, int N, int B, int n, int k,
    int nsub, int pk, int nsplit, float scale, int64_t R, int bh, int G)
{
    using C = F32Cfg<D>;
    using Ga = Gather<T, D>;
    constexpr int NW = C::NWF, LD = C::LD;
    extern __shared__ __align__(16) float sm[];
    const int tid = threadIdx.x, wave = tid / kWave, lane = tid % kWave, m16 = lane & 15, g = lane >> 4;
    float* sK = sm;
    float* sV = sK + 16 * NT * LD;
    float* stQ = sV + 16 * NT * LD + wave * 16 * LD;
    int s, u;                                               // slice, (key block, part, share of the walk)
    if (!schedule(blockIdx.x, bh, n * nsub * nsplit, s, u)) return;
    const int split = u % nsplit, jc = u / nsplit, j = jc / nsub, c = jc - j * nsub;
    const int own_first = c * pk, nk = min(pk, B - own_first);
    const int64_t sbase = (int64_t)s * N, kvbase = (int64_t)(s / G) * N;
    const int32_t* os = off + (int64_t)s * (n + 1);
    const int lo = os[j];
    Walk w;
    w.nlist = os[j + 1] - lo;
    w.src = w.nlist > 0 ? ql + (int64_t)s * R + lo : os;
    w.llast = max(w.nlist - 1, 0);
    w.own0 = j * B + own_first;
    w.own_e = k << 24;
    w.total = w.nlist + (B - own_first);
    stage_rows<T, D, 16 * NT, NW * kWave>(K + (kvbase + w.own0) * D, sK, nk, tid);
    __shared__ int odd[NW];                                 // of the V rows that each wave brought
    const bool mine = stage_rows<T, D, 16 * NT, NW * kWave>(V + (kvbase + w.own0) * D, sV, nk, tid);
    odd[wave] = __ballot(mine) != 0;
    __syncthreads();

    const float c2 = scale * kLog2e;
    const int64_t slots = (int64_t)(k + 1) * nsub;
    const int grow = lane / Ga::CPR, gcol = (lane % Ga::CPR) * Ga::EPL;
    const T* Qs = Q + sbase * D + gcol;
    const int32_t* kept = k > 0 ? idx + sbase * k : os;     // (k = 0: no rows; any readable address serves)
    // t: entries of the rows this lane gathers a piece of; tl: of row m16, there: what its row of kept blocks
    // holds at the entry's place
    auto ids = [&](int a0, int (&t)[Ga::NI], int& tl) {
#pragma unroll
        for (int i = 0; i < Ga::NI; ++i) t[i] = w.at(a0 + Ga::RPI * i + grow);
        tl = w.at(a0 + m16);
    };
    auto fetch = [&](const int (&t)[Ga::NI], int tl, u32x4_t (&q)[Ga::NI], int& there) {
#pragma unroll
        for (int i = 0; i < Ga::NI; ++i) q[i] = *reinterpret_cast<const u32x4_t*>(Qs + (int64_t)list_query(t[i]) * D);
        there = kept[(int64_t)list_query(tl) * k + min(list_slot(tl), max(k - 1, 0))];
    };
    const int stride = 16 * NW * nsplit;
    int a0 = 16 * (split * NW + wave);
    int tA[Ga::NI], tN[Ga::NI], tlA, tlN, thereA;
    u32x4_t qr[Ga::NI];
    ids(a0, tA, tlA);
    ids(a0 + stride, tN, tlN);
    fetch(tA, tlA, qr, thereA);
    for (; a0 < w.total; a0 += stride) {
        // park the 16 rows; the next step's loads go out
        const int tl = tlA, there = thereA;
#pragma unroll
        for (int i = 0; i < Ga::NI; ++i) put<T>(stQ + (grow + Ga::RPI * i) * LD + gcol, qr[i]);
#pragma unroll
        for (int i = 0; i < Ga::NI; ++i) tA[i] = tN[i];
        tlA = tlN;
        ids(a0 + 2 * stride, tN, tlN);
        fetch(tA, tlA, qr, thereA);
        __builtin_amdgcn_wave_barrier();
        // S^T: keys x queries.  Operands come from LDS one step ahead, here and below: 1 % at d = 64, 4 % at 128
        f32x4_t x[NT], qa[2], ka[2][NT];
#pragma unroll
        for (int kt = 0; kt < NT; ++kt) x[kt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int t = -1; t < C::MT; ++t) {
            if (t + 1 < C::MT) {
                qa[(t + 1) & 1] = *reinterpret_cast<const f32x4_t*>(stQ + m16 * LD + 16 * (t + 1) + 4 * g);
#pragma unroll
                for (int kt = 0; kt < NT; ++kt)
                    ka[(t + 1) & 1][kt] = *reinterpret_cast<const f32x4_t*>(sK + (16 * kt + m16) * LD + 16 * (t + 1) + 4 * g);
            }
            __builtin_amdgcn_sched_barrier(0);
            if (t >= 0) {
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int kt = 0; kt < NT; ++kt) x[kt] = mfma4(ka[t & 1][kt][i], qa[t & 1][i], x[kt]);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        // own row r sees keys 0 .. r of the part; keys beyond the part's do not exist
        const int av = a0 + m16, r = av < w.nlist ? nk - 1 : min(av - w.nlist, nk - 1);
        float mref = -INFINITY;
#pragma unroll
        for (int kt = 0; kt < NT; ++kt)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                x[kt][i] = 16 * kt + 4 * g + i <= r ? x[kt][i] * c2 : -INFINITY;
                mref = max_nan(mref, x[kt][i]);
            }
        mref = max_nan(mref, __shfl_xor(mref, 16, kWave));
        mref = max_nan(mref, __shfl_xor(mref, 32, kWave));
        float l = 0.f;
        const float ref = fmaxf(mref, -kFltLargest);             // (no finite logit in this part: no weight)
#pragma unroll
        for (int kt = 0; kt < NT; ++kt)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                x[kt][i] = fast_exp2(x[kt][i] - ref);
                l += x[kt][i];
            }
        l += __shfl_xor(l, 16, kWave);
        l += __shfl_xor(l, 32, kWave);
        // O^T = V^T P^T
        f32x4_t o[C::MT];
#pragma unroll
        for (int mt = 0; mt < C::MT; ++mt) o[mt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        f32x4_t va[2][C::H];
        auto value = [&](int r) {
#pragma unroll
            for (int h = 0; h < C::H; ++h)
                va[r & 1][h] = *reinterpret_cast<const f32x4_t*>(sV + (16 * (r / 4) + 4 * g + r % 4) * LD + 64 * h + 4 * m16);
        };
        value(0);
#pragma unroll
        for (int r = 0; r < 4 * NT; ++r) {
            if (r + 1 < 4 * NT) value(r + 1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int h = 0; h < C::H; ++h)
#pragma unroll
                for (int mt = 0; mt < 4; ++mt) o[4 * h + mt] = mfma4(va[r & 1][h][mt], x[r / 4][r % 4], o[4 * h + mt]);
            __builtin_amdgcn_sched_barrier(0);
        }
        // the partial: this lane holds channels 64 h + 16 g .. + 15 of its row
        // (clamped: lists that do not match the rows of kept blocks give a wrong result, never an address
        // outside the partials)
        const int e = place_of(tl, there, kept + (int64_t)list_query(tl) * k, j, k);
        if (av < w.total && e >= 0) {
            const int64_t prow = (sbase + min(list_query(tl), N - 1)) * slots + (int64_t)min(e, k) * nsub + c;
            float* dst = PO + prow * D + 16 * g;
#pragma unroll
            for (int h = 0; h < C::H; ++h)
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    *reinterpret_cast<f32x4_t*>(dst + 64 * h + 4 * i) =
                        f32x4_t{o[4 * h][i], o[4 * h + 1][i], o[4 * h + 2][i], o[4 * h + 3][i]};
            if (g == 0) Pml[prow] = make_float2(mref, l);
        }
        __builtin_amdgcn_wave_barrier();
    }
    int any = 0;
#pragma unroll
    for (int v = 0; v < NW; ++v) any |= odd[v];
    if (!any) return;
    OwnRows own(off, N, B, n, nsub, pk, nsplit, bh, G, NW);
    own.again([&](int t, int seen) {
        const float z = own.lane < seen ? scale * kLog2e * row_dot<T, D>(Q + (own.q0 + t) * D, K + (own.kv0 + own.lane) * D) : -INFINITY;
        const float top = wave_max(z), p = fast_exp2(z - fmaxf(top, -kFltLargest)), l = wave_sum(p);
        const int64_t prow = ((own.q0 + t) * (k + 1) + k) * nsub + own.c;
        weigh_rows<T, D>(p, seen, V + own.kv0 * D, sm + (2 * 16 * NT + own.wave * 16) * LD, PO + prow * D, own.lane);
        if (own.lane == 0) Pml[prow] = make_float2(top, l);
    });
}

// A query's partials, [kept block or own block][part]: which exist
struct Slots {
    int k, nsub, own_parts;
    __device__ __forceinline__ bool counts(const int32_t* irow, int e, int c) const
    {
        return e == k ? c < own_parts : irow[e] >= 0;
    }
};

// O_t = sum_p 2^(m_p - M) o_p / sum_p 2^(m_p - M) l_p, lse_t = (M + log2 L) ln 2; D / 4 lanes per query,
// partials in order, eight loads in flight
template <typename T, int D>
__global__ __launch_bounds__(256) void fwd_f32_merge_kernel(
    const int32_t* __restrict__ idx, const float* __restrict__ PO, const float2* __restrict__ Pml, T* __restrict__ O,
    float* __restrict__ lse, int N, int B, int k, int nsub, int pk, int64_t rows_total)
{
    constexpr int L = D / 4, CH = 8;
    const int64_t row = (int64_t)blockIdx.x * (256 / L) + threadIdx.x / L;
    const int part = threadIdx.x % L;
    if (row >= rows_total) return;
    const Slots sl = {k, nsub, (int)(row % N) % B / pk + 1};
    const int slots = (k + 1) * nsub;
    const int32_t* irow = idx + row * k;
    const float2* ml = Pml + row * slots;
    const float* po = PO + row * slots * D + 4 * part;
    float M = -INFINITY;
    for (int p = part; p < slots; p += L)                   // the lanes of a query share its partials out
        if (sl.counts(irow, p / nsub, p % nsub)) M = max_nan(M, ml[p].x);
    for (int o = 1; o < L; o <<= 1) M = max_nan(M, __shfl_xor(M, o, kWave));
    float Ls = 0.f;
    f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
    for (int p0 = 0; p0 < slots; p0 += CH) {
        float2 x[CH];
        f32x4_t v[CH];
        bool ok[CH];
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            const int p = min(p0 + i, slots - 1);
            ok[i] = p0 + i < slots && sl.counts(irow, p / nsub, p % nsub);
            x[i] = ml[p];
            v[i] = *reinterpret_cast<const f32x4_t*>(po + (int64_t)p * D);
        }
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            if (!ok[i]) continue;                           // (holds whatever the workspace held)
            const float wt = fast_exp2(x[i].x - M);
            Ls = fmaf(wt, x[i].y, Ls);
#pragma unroll
            for (int c = 0; c < 4; ++c) acc[c] = fmaf(wt, v[i][c], acc[c]);
        }
    }
    const float inv = 1.f / Ls;
#pragma unroll
    for (int c = 0; c < 4; ++c) O[row * D + 4 * part + c] = from_f32<T>(acc[c] * inv);
    if (part == 0) lse[row] = (M + fast_log2(Ls)) * kLn2;
}

// Backward: per step of 16 queries
//   S = Q K^T, dP = dO V^T - D        queries x keys, so that P and dS are operands over the queries
//   dV^T += dO^T P, dK^T += Q^T dS    channels x keys, kept in registers for the whole walk
//   dQ^T  = K^T dS^T                  dS turned over through LDS; written as a partial
// For parts of up to three 16-key tiles (d = 128: two), where bwd_f32_wide_kernel's waves would lack keys.
// want_dq / want_dkv: which results the caller asked for.  The dK and dV of a workgroup's waves are
// added up through LDS; with several shares of a walk or several query heads per key/value head they go
// to sums[dK | dV][query slice][share][N][D] and kv_sum_f32_kernel adds those up in order.
template <typename T, int D, int NT>
__global__ __launch_bounds__(F32Cfg<D>::NWB * kWave) void bwd_f32_km_kernel(
    const T* __restrict__ Q, const T* __restrict__ K, const T* __restrict__ V, const T* __restrict__ dO,
    const float2* __restrict__ ld, const int32_t* __restrict__ idx, const int32_t* __restrict__ off,
    const int32_t* __restrict__ ql, float* __restrict__ PdQ, T* __restrict__ dK, T* __restrict__ dV, float* __restrict__ sums, int N, int B, int n,
    int k, int nsub, int pk, int nsplit, float scale, int64_t R, int bh, int G, int want_dq, int want_dkv)
{
    using C = F32Cfg<D>;
    using Ga = Gather<T, D>;
    constexpr int NW = C::NWB, LD = C::LD, TL = 16 * NT + 4;
    extern __shared__ __align__(16) float sm[];
    const int tid = threadIdx.x, wave = tid / kWave, lane = tid % kWave, m16 = lane & 15, g = lane >> 4;
    float* sK = sm;
    float* sV = sK + 16 * NT * LD;
    float* stQ = sV + 16 * NT * LD + wave * C::bwd_wave_words(NT);
    float* stG = stQ + 16 * LD;
    float* sT = stG + 16 * LD;                              // dS of the step, [query][key]
    float* sl = sT + 16 * TL;                               // [16] lse log2 e, [16] -D
    int s, u;
    if (!schedule(blockIdx.x, bh, n * nsub * nsplit, s, u)) return;
    const int split = u % nsplit, jc = u / nsplit, j = jc / nsub, c = jc - j * nsub;
    const int own_first = c * pk, nk = min(pk, B - own_first);
    const int64_t sbase = (int64_t)s * N, kvbase = (int64_t)(s / G) * N;
    const int32_t* os = off + (int64_t)s * (n + 1);
    const int lo = os[j];
    Walk w;
    w.nlist = os[j + 1] - lo;
    w.src = w.nlist > 0 ? ql + (int64_t)s * R + lo : os;
    w.llast = max(w.nlist - 1, 0);
    w.own0 = j * B + own_first;
    w.own_e = k << 24;
    w.total = w.nlist + (B - own_first);
    __shared__ int odd[NW];                                 // of the rows that each wave brought
    bool mine = stage_rows<T, D, 16 * NT, NW * kWave>(K + (kvbase + w.own0) * D, sK, nk, tid);
    mine = stage_rows<T, D, 16 * NT, NW * kWave>(V + (kvbase + w.own0) * D, sV, nk, tid) || mine;
    odd[wave] = __ballot(mine) != 0;
    __syncthreads();

    const float c2 = scale * kLog2e;
    const int64_t slots = (int64_t)(k + 1) * nsub;
    const int grow = lane / Ga::CPR, gcol = (lane % Ga::CPR) * Ga::EPL;
    const T* Qs = Q + sbase * D + gcol;
    const T* Gs = dO + sbase * D + gcol;
    const int32_t* kept = k > 0 ? idx + sbase * k : os;     // (as in the forward, like `there` below)
    auto ids = [&](int a0, int (&t)[Ga::NI], int& tl) {
#pragma unroll
        for (int i = 0; i < Ga::NI; ++i) t[i] = w.at(a0 + Ga::RPI * i + grow);
        tl = w.at(a0 + m16);
    };
    auto fetch = [&](int a0, const int (&t)[Ga::NI], int tl, u32x4_t (&q)[Ga::NI], u32x4_t (&gr)[Ga::NI], float2& x,
                     int& there) {
#pragma unroll
        for (int i = 0; i < Ga::NI; ++i) {
            q[i] = *reinterpret_cast<const u32x4_t*>(Qs + (int64_t)list_query(t[i]) * D);
            gr[i] = *reinterpret_cast<const u32x4_t*>(Gs + (int64_t)list_query(t[i]) * D);
        }
        x = ld[sbase + list_query(tl)];
        there = kept[(int64_t)list_query(tl) * k + min(list_slot(tl), max(k - 1, 0))];
        if (a0 + m16 >= w.total) x = make_float2(INFINITY, 0.f);           // no such row: P = 0
    };
    f32x4_t dKT[C::MT][NT], dVT[C::MT][NT];
#pragma unroll
    for (int mt = 0; mt < C::MT; ++mt)
#pragma unroll
        for (int kt = 0; kt < NT; ++kt) {
            dKT[mt][kt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
            dVT[mt][kt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        }
    const int stride = 16 * NW * nsplit;
    int a0 = 16 * (split * NW + wave);
    int tA[Ga::NI], tN[Ga::NI], tlA, tlN, thereA;
    u32x4_t qr[Ga::NI], gr[Ga::NI];
    float2 xl;
    ids(a0, tA, tlA);
    ids(a0 + stride, tN, tlN);
    fetch(a0, tA, tlA, qr, gr, xl, thereA);
    for (; a0 < w.total; a0 += stride) {
        const int tl = tlA, there = thereA;
#pragma unroll
        for (int i = 0; i < Ga::NI; ++i) {
            float* row = stQ + (grow + Ga::RPI * i) * LD;
            put<T>(row + gcol, qr[i]);
            put<T>(row + 16 * LD + gcol, gr[i]);
        }
        if (lane < 16) { sl[lane] = xl.x; sl[16 + lane] = xl.y; }
#pragma unroll
        for (int i = 0; i < Ga::NI; ++i) tA[i] = tN[i];
        tlA = tlN;
        ids(a0 + 2 * stride, tN, tlN);
        fetch(a0 + stride, tA, tlA, qr, gr, xl, thereA);
        __builtin_amdgcn_wave_barrier();
        const f32x4_t l4 = *reinterpret_cast<const f32x4_t*>(sl + 4 * g);
        const f32x4_t nd = *reinterpret_cast<const f32x4_t*>(sl + 16 + 4 * g);
        f32x4_t x[NT], dp[NT];
#pragma unroll
        for (int kt = 0; kt < NT; ++kt) { x[kt] = f32x4_t{0.f, 0.f, 0.f, 0.f}; dp[kt] = nd; }
#pragma unroll
        for (int t = 0; t < C::MT; ++t) {
            const f32x4_t q = *reinterpret_cast<const f32x4_t*>(stQ + m16 * LD + 16 * t + 4 * g);
            const f32x4_t gq = *reinterpret_cast<const f32x4_t*>(stG + m16 * LD + 16 * t + 4 * g);
#pragma unroll
            for (int kt = 0; kt < NT; ++kt) {
                const f32x4_t a = *reinterpret_cast<const f32x4_t*>(sK + (16 * kt + m16) * LD + 16 * t + 4 * g);
                const f32x4_t b = *reinterpret_cast<const f32x4_t*>(sV + (16 * kt + m16) * LD + 16 * t + 4 * g);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    x[kt] = mfma4(q[i], a[i], x[kt]);
                    dp[kt] = mfma4(gq[i], b[i], dp[kt]);
                }
            }
        }
        // this lane: key 16 kt + m16 of the part, queries a0 + 4 g + i, which see the keys below `seen`
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int a = a0 + 4 * g + i, seen = a < w.nlist ? nk : min(a - w.nlist + 1, nk);
#pragma unroll
            for (int kt = 0; kt < NT; ++kt) {
                const float p = 16 * kt + m16 < seen ? fast_exp2(fmaf(x[kt][i], c2, -l4[i])) : 0.f;
                x[kt][i] = p;
                dp[kt][i] *= p;
            }
        }
        if (want_dq) {
#pragma unroll
            for (int kt = 0; kt < NT; ++kt)
#pragma unroll
                for (int i = 0; i < 4; ++i) sT[(4 * g + i) * TL + 16 * kt + m16] = dp[kt][i];
        }
        if (want_dkv) {
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int h = 0; h < C::H; ++h) {
                    const f32x4_t q = *reinterpret_cast<const f32x4_t*>(stQ + (4 * g + i) * LD + 64 * h + 4 * m16);
                    const f32x4_t gq = *reinterpret_cast<const f32x4_t*>(stG + (4 * g + i) * LD + 64 * h + 4 * m16);
#pragma unroll
                    for (int kt = 0; kt < NT; ++kt)
#pragma unroll
                        for (int mt = 0; mt < 4; ++mt) {
                            dVT[4 * h + mt][kt] = mfma4(gq[mt], x[kt][i], dVT[4 * h + mt][kt]);
                            dKT[4 * h + mt][kt] = mfma4(q[mt], dp[kt][i], dKT[4 * h + mt][kt]);
                        }
                }
        }
        if (want_dq) {
            __builtin_amdgcn_wave_barrier();
            f32x4_t o[C::MT];
#pragma unroll
            for (int mt = 0; mt < C::MT; ++mt) o[mt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kt = 0; kt < NT; ++kt) {
                const f32x4_t b = *reinterpret_cast<const f32x4_t*>(sT + m16 * TL + 16 * kt + 4 * g);
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int h = 0; h < C::H; ++h) {
                        const f32x4_t a = *reinterpret_cast<const f32x4_t*>(sK + (16 * kt + 4 * g + i) * LD + 64 * h + 4 * m16);
#pragma unroll
                        for (int mt = 0; mt < 4; ++mt) o[4 * h + mt] = mfma4(a[mt], b[i], o[4 * h + mt]);
                    }
            }
            const int e = place_of(tl, there, kept + (int64_t)list_query(tl) * k, j, k);
            if (a0 + m16 < w.total && e >= 0) {
                const int64_t prow = (sbase + min(list_query(tl), N - 1)) * slots + (int64_t)min(e, k) * nsub + c;
                float* dst = PdQ + prow * D + 16 * g;
#pragma unroll
                for (int h = 0; h < C::H; ++h)
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        *reinterpret_cast<f32x4_t*>(dst + 64 * h + 4 * i) =
                            f32x4_t{o[4 * h][i], o[4 * h + 1][i], o[4 * h + 2][i], o[4 * h + 3][i]};
            }
        }
        __builtin_amdgcn_wave_barrier();
    }
    int any = 0;
#pragma unroll
    for (int v = 0; v < NW; ++v) any |= odd[v];
    if (want_dkv) {
        // sum over the waves, in order, through LDS: over the K and V tiles (row-major, keys x channels)
        __syncthreads();
        for (int wv = 0; wv < NW; ++wv) {
            if (wave == wv) {
#pragma unroll
                for (int kt = 0; kt < NT; ++kt)
#pragma unroll
                    for (int h = 0; h < C::H; ++h)
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            // result rows 4 g + i of tile 4 h + mt: channel 64 h + 16 g + 4 i + mt of key 16 kt + m16
                            float* pk_ = sK + (16 * kt + m16) * LD + 64 * h + 16 * g + 4 * i;
                            float* pv_ = sV + (16 * kt + m16) * LD + 64 * h + 16 * g + 4 * i;
                            f32x4_t a = {dKT[4 * h][kt][i], dKT[4 * h + 1][kt][i], dKT[4 * h + 2][kt][i], dKT[4 * h + 3][kt][i]};
                            f32x4_t b = {dVT[4 * h][kt][i], dVT[4 * h + 1][kt][i], dVT[4 * h + 2][kt][i], dVT[4 * h + 3][kt][i]};
                            if (wv > 0) {
                                a += *reinterpret_cast<const f32x4_t*>(pk_);
                                b += *reinterpret_cast<const f32x4_t*>(pv_);
                            }
                            *reinterpret_cast<f32x4_t*>(pk_) = a;
                            *reinterpret_cast<f32x4_t*>(pv_) = b;
                        }
            }
            __syncthreads();
        }
        for (int i = tid; i < 2 * nk * (D / 4); i += NW * kWave) {
            const int which = i / (nk * (D / 4)), rem = i % (nk * (D / 4)), key = rem / (D / 4), ch = 4 * (rem % (D / 4));
            f32x4_t v = *reinterpret_cast<const f32x4_t*>((which == 0 ? sK : sV) + key * LD + ch);
            if (which == 0) v *= scale;
            const int64_t at = w.own0 + key;
            if (sums) {
                *reinterpret_cast<f32x4_t*>(sums + ((((int64_t)which * bh + s) * nsplit + split) * N + at) * D + ch) = v;
            } else {
                T* dst = (which == 0 ? dK : dV) + (kvbase + at) * D + ch;
#pragma unroll
                for (int e = 0; e < 4; ++e) dst[e] = from_f32<T>(v[e]);
            }
        }
    }
    if (!any || !want_dq) return;
    OwnRows own(off, N, B, n, nsub, pk, nsplit, bh, G, NW);
    own.again([&](int t, int seen) {
        float ds = 0.f;
        if (own.lane < seen) {
            const int64_t key = (own.kv0 + own.lane) * D;
            const float2 x = ld[own.q0 + t];
            const float z = scale * kLog2e * row_dot<T, D>(Q + (own.q0 + t) * D, K + key);
            ds = fast_exp2(z - x.x) * (row_dot<T, D>(dO + (own.q0 + t) * D, V + key) + x.y);
        }
        weigh_rows<T, D>(ds, seen, K + own.kv0 * D, sm + 2 * 16 * NT * LD + own.wave * C::bwd_wave_words(NT),
                         PdQ + (((own.q0 + t) * (k + 1) + k) * nsub + own.c) * D, own.lane);
    });
}

// Backward for parts of four 16-key tiles: a wave of four owns one tile and keeps what it needs of K and V in registers, as
// matrix operands, for the whole walk: K and V of its keys for S and dP, K of all keys for its share of dQ's channels.  LDS
// only holds the gathered rows, which all waves read, and dS, on its way from the waves of the keys to the waves of the
// channels; both twice, so that a step of RQ queries has one barrier:
//   S, dP -> dS to LDS; dV^T, dK^T; the next step's rows to LDS | barrier | dQ^T = K^T dS^T over all keys, a partial
// The kernel above, whose waves take 16 queries against all keys each, kept 128 sums a wave, had room for eight waves on a compute
// unit, and added its waves' sums up one after the other at the end, as much work as the two steps that a wave had between: at the
// shape above 167 us (1024 workgroups of eight waves) against 123 (1536 of four), whole step 300 -> 244; 2 x 8 heads of 8192,
// d = 128, B = 64, k = 8 2309 -> 1875 (there it could take 32 keys, so that dQ had twice the partials).
// Three waves per SIMD leave 168 registers at d = 64, fp32, and the walk just fits them (one value is stored before it and read after it):
// with six values spilled in every step the shape's backward, all of it, took 154 us instead of 147, 16 slices of 8192 552 instead of 519.
template <int D>
struct WideCfg {
    static constexpr int QT = D == 64 ? 2 : 1, RQ = 16 * QT;      // 16-query tiles, queries per step
    static constexpr int NW = 4, LD = D + 4, TL = 64 + 4, WPS = D == 64 ? 3 : 2;
    static constexpr int words = 4 * RQ * LD + 2 * RQ * TL + 2 * 3 * RQ;
    static constexpr size_t lds = sizeof(float) * words;
};

template <typename T>
__device__ __forceinline__ f32x4_t four(const T* p)
{
    if constexpr (sizeof(T) == 4) {
        return *reinterpret_cast<const f32x4_t*>(p);
    } else {
        const uint2 x = *reinterpret_cast<const uint2*>(p);
        return f32x4_t{__uint_as_float(x.x << 16), __uint_as_float(x.x & 0xffff0000u), __uint_as_float(x.y << 16),
                       __uint_as_float(x.y & 0xffff0000u)};
    }
}

template <typename T, int D>
__global__ __launch_bounds__(WideCfg<D>::NW * kWave, WideCfg<D>::WPS) void bwd_f32_wide_kernel(
    const T* __restrict__ Q, const T* __restrict__ K, const T* __restrict__ V, const T* __restrict__ dO,
    const float2* __restrict__ ld, const int32_t* __restrict__ idx, const int32_t* __restrict__ off,
    const int32_t* __restrict__ ql, float* __restrict__ PdQ, T* __restrict__ dK, T* __restrict__ dV, float* __restrict__ sums, int N, int B, int n,
    int k, int nsub, int pk, int nsplit, float scale, int64_t R, int bh, int G, int want_dq, int want_dkv)
{
    using C = WideCfg<D>;
    using Ga = Gather<T, D>;
    constexpr int NW = C::NW, LD = C::LD, TL = C::TL, QT = C::QT, RQ = C::RQ, MT = D / 16, H = D / 64;
    constexpr int RPP = NW * kWave / Ga::CPR, NI = RQ / RPP;      // rows that the workgroup gathers at once, how often
    static_assert(NI * RPP == RQ, "");
    extern __shared__ __align__(16) float sm[];
    const int tid = threadIdx.x, lane = tid % kWave, m16 = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    float* const sT = sm + 4 * RQ * LD;                           // dS of a step, [query][key]
    float* const sl = sT + 2 * RQ * TL;                           // [RQ] lse log2 e, [RQ] -D, [RQ] row of the partial
    int s, u;
    if (!schedule(blockIdx.x, bh, n * nsub * nsplit, s, u)) return;
    const int split = u % nsplit, jc = u / nsplit, j = jc / nsub, c = jc - j * nsub;
    const int own_first = c * pk, nk = min(pk, B - own_first);
    const int64_t sbase = (int64_t)s * N, kvbase = (int64_t)(s / G) * N;
    const int32_t* os = off + (int64_t)s * (n + 1);
    const int lo = os[j];
    Walk w;
    w.nlist = os[j + 1] - lo;
    w.src = w.nlist > 0 ? ql + (int64_t)s * R + lo : os;
    w.llast = max(w.nlist - 1, 0);
    w.own0 = j * B + own_first;
    w.own_e = k << 24;
    w.total = w.nlist + (B - own_first);

    const float c2 = scale * kLog2e;
    const int slots = (k + 1) * nsub;
    const int grow = tid / Ga::CPR, gcol = (tid % Ga::CPR) * Ga::EPL;
    Q += sbase * D;
    dO += sbase * D;
    const int32_t* kept = k > 0 ? idx + sbase * k : os;     // (as in the forward, like `there` below)
    // t: entries of the rows that this thread gathers a piece of; tl (the first RQ threads): of row tid
    auto ids = [&](int a0, int (&t)[NI], int& tl) {
#pragma unroll
        for (int i = 0; i < NI; ++i) t[i] = w.at(a0 + RPP * i + grow);
        if (tid < RQ) tl = w.at(a0 + tid);
    };
    u32x4_t qr[NI], gr[NI];
    float2 xl = make_float2(INFINITY, 0.f);
    int tA[NI], tN[NI], tlA = 0, tlN = 0, there = 0;
    auto fetch = [&](int a0) {
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int64_t o = (int64_t)list_query(tA[i]) * D + gcol;   // (pointers of a lane's own would be two registers more each)
            qr[i] = *reinterpret_cast<const u32x4_t*>(Q + o);
            gr[i] = *reinterpret_cast<const u32x4_t*>(dO + o);
        }
        if (tid < RQ) {
            xl = ld[sbase + list_query(tlA)];
            there = kept[(int64_t)list_query(tlA) * k + min(list_slot(tlA), max(k - 1, 0))];
        }
    };
    // the rows of the step at a0, which have been requested, to buffer b; the requests for the step after it
    const int stride = RQ * nsplit;
    auto park = [&](int a0, int b) {
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            float* row = sm + (2 * b * RQ + grow + RPP * i) * LD + gcol;
            put<T>(row, qr[i]);
            put<T>(row + RQ * LD, gr[i]);
        }
        if (tid < RQ) {
            const bool live = a0 + tid < w.total;
            float* x = sl + 3 * b * RQ + tid;
            x[0] = live ? xl.x : INFINITY;                  // (no such row: P = 0)
            x[RQ] = live ? xl.y : 0.f;
            // clamped as in the forward; the partials number less than 2^31 (f32_km_path)
            const int e = place_of(tlA, there, kept + (int64_t)list_query(tlA) * k, j, k);
            const int prow = (int)((sbase + min(list_query(tlA), N - 1)) * slots) + min(e, k) * nsub + c;
            reinterpret_cast<int*>(x)[2 * RQ] = live && e >= 0 ? prow : -1;
        }
#pragma unroll
        for (int i = 0; i < NI; ++i) tA[i] = tN[i];
        tlA = tlN;
        ids(a0 + 2 * stride, tN, tlN);
        fetch(a0 + stride);
    };
    int a0 = RQ * split;
    ids(a0, tA, tlA);
    ids(a0 + stride, tN, tlN);

    // operands: keys 16 wave + m16 of the part, channels 16 t + 4 g ..; keys 16 kt + 4 g + i, channel 16 (H wave + h) + m16
    f32x4_t kop[MT], vop[MT], kq[4][H];
    {
        const int key = 16 * wave + m16;
        const int64_t row = (kvbase + w.own0 + min(key, nk - 1)) * D + 4 * g;
#pragma unroll
        for (int t = 0; t < MT; ++t) {
            kop[t] = four<T>(K + row + 16 * t);
            vop[t] = four<T>(V + row + 16 * t);
        }
#pragma unroll
        for (int kt = 0; kt < 4; ++kt)
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int h = 0; h < H; ++h)
                    kq[kt][h][i] = to_f32<T>(K[(kvbase + w.own0 + min(16 * kt + 4 * g + i, nk - 1)) * D + 16 * (H * wave + h) + m16]);
    }
    fetch(a0);
    __shared__ int odd[NW];                                 // of the rows of a wave
    {
        uint32_t top = 0u;
        const bool live = 16 * wave + m16 < nk;
#pragma unroll
        for (int t = 0; t < MT; ++t)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (!live) kop[t][i] = vop[t][i] = 0.f;
                top = max(top, max(__float_as_uint(kop[t][i]) & 0x7fffffffu, __float_as_uint(vop[t][i]) & 0x7fffffffu));
            }
        odd[wave] = __ballot(top >= 0x7f800000u) != 0;
#pragma unroll
        for (int kt = 0; kt < 4; ++kt)
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int h = 0; h < H; ++h) kq[kt][h][i] = 16 * kt + 4 * g + i < nk ? kq[kt][h][i] : 0.f;
    }
    f32x4_t dKT[MT], dVT[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) dKT[mt] = dVT[mt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    park(a0, 0);
    __syncthreads();
    for (int b = 0; a0 < w.total; a0 += stride, b ^= 1) {
        const float* stQ = sm + 2 * b * RQ * LD;
        const float* stG = stQ + RQ * LD;
        float* stT = sT + b * RQ * TL;
        const float* xb = sl + 3 * b * RQ;
        f32x4_t x[QT], dp[QT];
#pragma unroll
        for (int q = 0; q < QT; ++q) {
            x[q] = f32x4_t{0.f, 0.f, 0.f, 0.f};
            dp[q] = *reinterpret_cast<const f32x4_t*>(xb + RQ + 16 * q + 4 * g);
        }
#pragma unroll
        for (int t = 0; t < MT; ++t) {
            f32x4_t qv[QT], gv[QT];
#pragma unroll
            for (int q = 0; q < QT; ++q) {
                qv[q] = *reinterpret_cast<const f32x4_t*>(stQ + (16 * q + m16) * LD + 16 * t + 4 * g);
                gv[q] = *reinterpret_cast<const f32x4_t*>(stG + (16 * q + m16) * LD + 16 * t + 4 * g);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int q = 0; q < QT; ++q) {
                    x[q] = mfma4(qv[q][i], kop[t][i], x[q]);
                    dp[q] = mfma4(gv[q][i], vop[t][i], dp[q]);
                }
        }
        // this lane: key 16 wave + m16 of the part, queries a0 + 16 q + 4 g + i, which see the keys below `seen`
#pragma unroll
        for (int q = 0; q < QT; ++q) {
            const f32x4_t l4 = *reinterpret_cast<const f32x4_t*>(xb + 16 * q + 4 * g);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int a = a0 + 16 * q + 4 * g + i, seen = a < w.nlist ? nk : min(a - w.nlist + 1, nk);
                const float p = 16 * wave + m16 < seen ? fast_exp2(fmaf(x[q][i], c2, -l4[i])) : 0.f;
                x[q][i] = p;
                dp[q][i] *= p;
                if (want_dq) stT[(16 * q + 4 * g + i) * TL + 16 * wave + m16] = dp[q][i];
            }
        }
        if (want_dkv) {
            // (the sums of sixteen queries first, then the walk's: one chain over all of a walk's queries is 5 % further from 64 bits than
            // the waves of bwd_f32_km_kernel, which share them out; so it is no further: dK of 4096 queries, k = 7 4.71e-7, now 4.47e-7, there
            // 4.50e-7; for 32 queries at a time 4.51e-7 and, of 2048, B = 128, k = 3, 4.19e-7 against 4.15e-7, and 1 to 2 % less time)
            auto add = [&](const float* rows, const f32x4_t (&y)[QT], f32x4_t (&acc)[MT]) {
#pragma unroll
                for (int h = 0; h < H; ++h) {
#pragma unroll
                    for (int q = 0; q < QT; ++q) {
                        f32x4_t z[4];
#pragma unroll
                        for (int mt = 0; mt < 4; ++mt) z[mt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const f32x4_t v = *reinterpret_cast<const f32x4_t*>(rows + (16 * q + 4 * g + i) * LD + 64 * h + 4 * m16);
#pragma unroll
                            for (int mt = 0; mt < 4; ++mt) z[mt] = mfma4(v[mt], y[q][i], z[mt]);
                        }
#pragma unroll
                        for (int mt = 0; mt < 4; ++mt) acc[4 * h + mt] += z[mt];
                    }
                }
            };
            add(stG, x, dVT);
            add(stQ, dp, dKT);
        }
        park(a0 + stride, b ^ 1);
        int prow[QT];                                       // (before the barrier: the step after it parks the next but one's rows there)
#pragma unroll
        for (int q = 0; q < QT; ++q) prow[q] = reinterpret_cast<const int*>(xb)[2 * RQ + 16 * q + m16];
        __syncthreads();
        if (want_dq) {
            f32x4_t o[QT][H], half[QT][H];                  // (d = 128: of 32 keys each)
#pragma unroll
            for (int q = 0; q < QT; ++q)
#pragma unroll
                for (int h = 0; h < H; ++h) o[q][h] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kt = 0; kt < 4; ++kt) {
                if (D == 128 && kt == 2) {
#pragma unroll
                    for (int q = 0; q < QT; ++q)
#pragma unroll
                        for (int h = 0; h < H; ++h) { half[q][h] = o[q][h]; o[q][h] = f32x4_t{0.f, 0.f, 0.f, 0.f}; }
                }
                f32x4_t ds[QT];
#pragma unroll
                for (int q = 0; q < QT; ++q) ds[q] = *reinterpret_cast<const f32x4_t*>(stT + (16 * q + m16) * TL + 16 * kt + 4 * g);
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int q = 0; q < QT; ++q)
#pragma unroll
                        for (int h = 0; h < H; ++h) o[q][h] = mfma4(kq[kt][h][i], ds[q][i], o[q][h]);
            }
            if constexpr (D == 128) {
#pragma unroll
                for (int q = 0; q < QT; ++q)
#pragma unroll
                    for (int h = 0; h < H; ++h) o[q][h] += half[q][h];
            }
#pragma unroll
            for (int q = 0; q < QT; ++q)
                if (prow[q] >= 0) {
#pragma unroll
                    for (int h = 0; h < H; ++h)
                        *reinterpret_cast<f32x4_t*>(PdQ + (int64_t)prow[q] * D + 16 * (H * wave + h) + 4 * g) = o[q][h];
                }
        }
    }
    if (want_dkv && 16 * wave + m16 < nk) {
        // result rows 4 g + i of tile 4 h + mt: channel 64 h + 16 g + 4 i + mt of key 16 wave + m16
        const int64_t at = w.own0 + 16 * wave + m16;
#pragma unroll
        for (int h = 0; h < H; ++h)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int ch = 64 * h + 16 * g + 4 * i;
                const f32x4_t a = f32x4_t{dKT[4 * h][i], dKT[4 * h + 1][i], dKT[4 * h + 2][i], dKT[4 * h + 3][i]} * scale;
                const f32x4_t v = {dVT[4 * h][i], dVT[4 * h + 1][i], dVT[4 * h + 2][i], dVT[4 * h + 3][i]};
                if (sums) {
                    float* dst = sums + (((int64_t)s * nsplit + split) * N + at) * D + ch;
                    *reinterpret_cast<f32x4_t*>(dst) = a;
                    *reinterpret_cast<f32x4_t*>(dst + (int64_t)bh * nsplit * N * D) = v;
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        dK[(kvbase + at) * D + ch + e] = from_f32<T>(a[e]);
                        dV[(kvbase + at) * D + ch + e] = from_f32<T>(v[e]);
                    }
                }
            }
    }
    int any = 0;
#pragma unroll
    for (int v = 0; v < NW; ++v) any |= odd[v];
    if (!any || !want_dq) return;
    __threadfence();                                        // (a row's partial is all waves' work)
    __syncthreads();
    if (wave >= QT) return;
    OwnRows own(off, N, B, n, nsub, pk, nsplit, bh, G, QT);
    own.again([&](int t, int seen) {
        float ds = 0.f;
        if (own.lane < seen) {
            const int64_t key = (own.kv0 + own.lane) * D;
            const float2 x = ld[own.q0 + t];
            const float z = scale * kLog2e * row_dot<T, D>(Q + (int64_t)t * D, K + key);
            ds = fast_exp2(z - x.x) * (row_dot<T, D>(dO + (int64_t)t * D, V + key) + x.y);
        }
        weigh_rows<T, D>(ds, seen, K + own.kv0 * D, sm + own.wave * kWave,
                         PdQ + (((own.q0 + t) * (k + 1) + k) * nsub + own.c) * D, own.lane);
    });
}

// dK, dV of a key/value slice = its sums over shares of the walk and query heads, in order
template <typename T>
__global__ __launch_bounds__(256) void kv_sum_f32_kernel(const float* __restrict__ sums, T* __restrict__ dK,
                                                         T* __restrict__ dV, int64_t quads_per_slice, int bhk, int terms)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x, per = quads_per_slice * bhk;
    if (i >= 2 * per) return;
    const int which = (int)(i / per);
    const int64_t r = i % per, skv = r / quads_per_slice, q = r % quads_per_slice;
    f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
    for (int t = 0; t < terms; ++t)
        acc += *reinterpret_cast<const f32x4_t*>(sums + ((((int64_t)which * bhk + skv) * terms + t) * quads_per_slice + q) * 4);
    T* dst = (which == 0 ? dK : dV) + r * 4;
#pragma unroll
    for (int e = 0; e < 4; ++e) dst[e] = from_f32<T>(acc[e]);
}

// dQ_t = scale * sum of its partials, in order
template <typename T, int D>
__global__ __launch_bounds__(256) void dq_f32_merge_kernel(const int32_t* __restrict__ idx, const float* __restrict__ PdQ,
                                                           T* __restrict__ dQ, int N, int B, int k, int nsub, int pk,
                                                           float scale, int64_t rows_total)
{
    constexpr int L = D / 4, CH = 8;
    const int64_t row = (int64_t)blockIdx.x * (256 / L) + threadIdx.x / L;
    const int part = threadIdx.x % L;
    if (row >= rows_total) return;
    const Slots sl = {k, nsub, (int)(row % N) % B / pk + 1};
    const int slots = (k + 1) * nsub;
    const int32_t* irow = idx + row * k;
    const float* po = PdQ + row * slots * D + 4 * part;
    f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
    for (int p0 = 0; p0 < slots; p0 += CH) {
        f32x4_t v[CH];
        bool ok[CH];
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            const int p = min(p0 + i, slots - 1);
            ok[i] = p0 + i < slots && sl.counts(irow, p / nsub, p % nsub);
            v[i] = *reinterpret_cast<const f32x4_t*>(po + (int64_t)p * D);
        }
#pragma unroll
        for (int i = 0; i < CH; ++i)
            if (ok[i]) acc += v[i];
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) dQ[row * D + 4 * part + c] = from_f32<T>(acc[c] * scale);
}

// ---- shapes, workspaces, launches --------------------------------------------------------------

namespace {

struct Cut {
    int nsub, pk, nt;            // parts per block, keys per part, 16-key tiles per part
};

// parts of equal size, at most `cap` keys
Cut cut_of(const Dims& s, int cap)
{
    Cut c;
    c.nsub = (s.B + cap - 1) / cap;
    c.pk = ((s.B + c.nsub - 1) / c.nsub + 15) / 16 * 16;
    c.nsub = (s.B + c.pk - 1) / c.pk;
    c.nt = c.pk / 16;
    return c;
}
Cut fwd_cut(const Dims& s) { return cut_of(s, 64); }
// backward: four tiles go to bwd_f32_wide_kernel; the other kernel has registers for the dK and dV of 48 keys (d = 128: 32)
bool bwd_wide(const Dims& s) { return cut_of(s, 64).nt == 4; }
Cut bwd_cut(const Dims& s) { return cut_of(s, s.D == 64 || bwd_wide(s) ? 64 : 32); }

size_t partials(const Dims& s, const Cut& c) { return (size_t)s.bh * s.N * (size_t)(s.k + 1) * c.nsub; }

// Steps of `rows` queries in a walk of average length
int64_t steps(const Dims& s, int rows) { return ((int64_t)(s.k + 1) * s.B + rows - 1) / rows; }

// Shares a walk is cut into, bwd_f32_km_kernel: about four workgroups per compute unit, at least one step of all waves each
int few_shares(const Dims& s, const Cut& c, int rows)
{
    const int64_t wgs = (int64_t)s.bh * s.n * c.nsub, want = (1024 + wgs - 1) / wgs;
    return (int)std::min(want, steps(s, rows));
}

// The others: the number with the least estimated time, in rows of a walk.  A launch takes what its `places` (three workgroups on a
// compute unit) have to do, `fixed` rows more per workgroup for its keys and values, its fill and the sums of dK and dV, or what is left
// when its longest walk begins and that walk, whose rows count `tail` of the average (they have a place to themselves in the end).  The longest
// walks are those of a slice's first blocks, B min(1, k / t) rows of the query blocks t = 1, 2, ...: they begin first, or, where the number of slices
// is a multiple of 8, with their XCD's last slice (schedule()).  The fourth powers round the corner between the two.
// Measured with one to 32 shares at 8 to 6144 walks, B = 16 to 4096, k = 0 to 20, which tail, fixed and places are fitted to: the number taken is
// about 1 % slower than the best on average (backward, d = 128: 3 %, for the two shares that bwd_shares() keeps); 1280 workgroups at least, and
// two shares up to 3072 walks, were 2 to 5 %.  Figures beside the calls.
int shares(const Dims& s, const Cut& c, int64_t most, double tail, double fixed, double places = 768.)
{
    const double walks = (double)s.bh * s.n * c.nsub, kept = std::min(s.k, s.n - 1);
    const double rows = (double)(s.k + 1) * s.B, longest = s.B * (1. + kept + kept * std::log(s.n / (kept + 1.)));
    const double before = s.bh % kXcds == 0 ? 1. - (double)kXcds / s.bh : 0.;      // of a launch, when the last slices begin
    auto time = [&](int ns) {
        const double all = walks / places * (rows + fixed * ns), last = before * all + tail * (longest / ns + fixed);
        return all * all * all * all + last * last * last * last;
    };
    int ns = 1;
    for (double t = time(1), more; ns < most && (more = time(ns + 1)) < t; ++ns) t = more;
    return ns;
}

bool sums_needed(const Dims& s, int nsplit) { return s.G * nsplit > 1; }

}  // namespace

// Everything the bf16 MFMA kernels do not cover, except: blocks too short for a 16-key tile to pay
// (fewer than 8 keys), rows of more than 64 kept blocks (a list entry holds the place in 8 bits), and
// shapes whose partial rows would take more than 16 GiB.  Those stay on the plain kernels.
bool f32_km_path(const Dims& s)
{
    return !mfma_path(s) && !(s.flags & MOBA_FLAG_REFERENCE_KERNELS) && s.B >= 8 && s.k <= kKeyMajorMaxTopk &&
           partials(s, cut_of(s, s.D == 64 ? 64 : 32)) * s.D * sizeof(float) <= ((size_t)16 << 30);
}

size_t forward_f32_km_ws_bytes(const Dims& s)
{
    const size_t p = partials(s, fwd_cut(s));
    return a256(p * s.D * sizeof(float)) + a256(p * sizeof(float2));
}

// [D: bh*N][(lse log2 e, -D): bh*N][partial dQ][sums of dK and dV]
size_t backward_f32_km_ld_offset(const Dims& s) { return a256(sizeof(float) * (size_t)s.bh * s.N); }
static size_t bwd_partials_offset(const Dims& s)
{
    return backward_f32_km_ld_offset(s) + a256(sizeof(float2) * (size_t)s.bh * s.N);
}
static size_t bwd_sums_offset(const Dims& s)
{
    return bwd_partials_offset(s) + a256(partials(s, bwd_cut(s)) * s.D * sizeof(float));
}
static int bwd_shares(const Dims& s)
{
    const Cut c = bwd_cut(s);
    if (!bwd_wide(s)) return few_shares(s, c, 16 * (s.D == 64 ? F32Cfg<64>::NWB : F32Cfg<128>::NWB));
    // us, shares of 1280 workgroups (two up to 3072 walks) -> these, B = 64: d = 64, 2 slices of 32768, k = 8 377 -> 329; 24 of 8192, k = 7 875 -> 818;
    // 6 of 8192 247 -> 224; d = 128, 12 of 2048, k = 2 127 -> 120.  Sixteen at most: 8 walks of 512 rows, d = 128, take 31 us, in 32 shares 38, and
    // the chain of sums over shares would cost more precision than shorter walks gain.  Two up to 3072 walks also where one is faster, for the
    // same reason: 20 slices of 4096, k = 2, dK 4.22e-7 from 64 bits in two shares, 4.25e-7 in one, which takes 20 % less.
    const int64_t most = std::min<int64_t>(16, steps(s, s.D == 64 ? WideCfg<64>::RQ : WideCfg<128>::RQ));
    const int ns = s.D == 64 ? shares(s, c, most, 0.8, 80.) : shares(s, c, most, 0.6, 80.);
    return (int64_t)s.bh * s.n * c.nsub < 3072 ? std::max(ns, (int)std::min<int64_t>(2, most)) : ns;
}
size_t backward_f32_km_ws_bytes(const Dims& s)
{
    const int ns = bwd_shares(s);
    return bwd_sums_offset(s) + (sums_needed(s, ns) ? a256(2 * sizeof(float) * (size_t)s.bh * ns * s.N * s.D) : 0);
}

template <typename T, int D, int NT>
static hipError_t fwd_launch_nt(const Dims& s, const Cut& c, const void* Q, const void* K, const void* V,
                                const int32_t* idx, const int32_t* off, const int32_t* ql, float* PO, float2* Pml,
                                void* O, float* lse, hipStream_t st)
{
    using C = F32Cfg<D>;
    // Shorter parts take less to begin with, and at d = 128 leave room for more workgroups.  us, shares of 1280 workgroups (d = 64: two up to
    // 3072 walks) -> these, B = 64: d = 64, 20 slices of 8192, k = 2 155 -> 141; 36 of 4096, k = 4 196 -> 181; 24 of 8192, k = 7 408 -> 382; d = 128,
    // 8 of 8192, k = 7 298 -> 277; 28 of 2048, k = 2 127 -> 114.
    const double part = std::sqrt(NT / 4.);
    const int ns = D == 64 ? shares(s, c, steps(s, 16 * C::NWF), 0.6, 56. * part)
                           : shares(s, c, steps(s, 16 * C::NWF), 0.3, 80. * part, 768. / part);
    hipError_t e = ensure_dynamic_lds((const void*)fwd_f32_km_kernel<T, D, NT>, C::fwd_lds(NT));
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((fwd_f32_km_kernel<T, D, NT>), dim3((unsigned)schedule_grid(s.bh, s.n * c.nsub * ns)),
                       dim3(C::NWF * kWave), C::fwd_lds(NT), st, (const T*)Q, (const T*)K, (const T*)V, idx, off, ql, PO, Pml,
                       s.N, s.B, s.n, s.k, c.nsub, c.pk, ns, s.scale, s.R, s.bh, s.G);
    const int64_t rows = (int64_t)s.bh * s.N;
    const int rpw = 256 / (D / 4);
    hipLaunchKernelGGL((fwd_f32_merge_kernel<T, D>), dim3((unsigned)((rows + rpw - 1) / rpw)), dim3(256), 0, st, idx, PO,
                       Pml, (T*)O, lse, s.N, s.B, s.k, c.nsub, c.pk, rows);
    return hipGetLastError();
}

template <typename T, int D, int NT>                       // NT: 4 for bwd_f32_wide_kernel
static hipError_t bwd_launch_nt(const Dims& s, const Cut& c, const void* Q, const void* K, const void* V, const void* dO,
                                const float2* ld, const int32_t* idx, const int32_t* off, const int32_t* ql, float* PdQ,
                                float* sums, void* dQ, void* dK, void* dV, uint32_t parts, hipStream_t st)
{
    const int ns = bwd_shares(s);
    const int want_dq = (parts & MOBA_BWD_DQ) != 0, want_dkv = (parts & MOBA_BWD_DKDV) != 0;
    auto go = [&](auto* kernel, int threads, size_t lds) {
        const hipError_t e = ensure_dynamic_lds((const void*)kernel, lds);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(kernel, dim3((unsigned)schedule_grid(s.bh, s.n * c.nsub * ns)), dim3(threads), lds, st,
                           (const T*)Q, (const T*)K, (const T*)V, (const T*)dO, ld, idx, off, ql, PdQ, (T*)dK, (T*)dV, sums,
                           s.N, s.B, s.n, s.k, c.nsub, c.pk, ns, s.scale, s.R, s.bh, s.G, want_dq, want_dkv);
        return hipSuccess;
    };
    hipError_t e;
    if constexpr (NT == 4) {
        e = go(bwd_f32_wide_kernel<T, D>, WideCfg<D>::NW * kWave, WideCfg<D>::lds);
    } else {
        e = go(bwd_f32_km_kernel<T, D, NT>, F32Cfg<D>::NWB * kWave, F32Cfg<D>::bwd_lds(NT));
    }
    if (e != hipSuccess) return e;
    if (want_dkv && sums) {
        const int64_t quads = (int64_t)s.N * D / 4, total = 2 * quads * s.bhk;
        hipLaunchKernelGGL(kv_sum_f32_kernel<T>, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, sums, (T*)dK,
                           (T*)dV, quads, s.bhk, s.G * ns);
    }
    if (want_dq) {
        const int64_t rows = (int64_t)s.bh * s.N;
        const int rpw = 256 / (D / 4);
        hipLaunchKernelGGL((dq_f32_merge_kernel<T, D>), dim3((unsigned)((rows + rpw - 1) / rpw)), dim3(256), 0, st, idx,
                           PdQ, (T*)dQ, s.N, s.B, s.k, c.nsub, c.pk, s.scale, rows);
    }
    return hipGetLastError();
}

hipError_t launch_forward_f32_km(const Dims& s, const void* Q, const void* K, const void* V, void* ws,
                                 const int32_t* idx, const int32_t* off, const int32_t* ql, void* O, float* lse,
                                 hipStream_t st)
{
    const Cut c = fwd_cut(s);
    float* PO = static_cast<float*>(ws);
    float2* Pml = reinterpret_cast<float2*>(static_cast<char*>(ws) + a256(partials(s, c) * s.D * sizeof(float)));
#define MOBA_F32(T, D, NT) return fwd_launch_nt<T, D, NT>(s, c, Q, K, V, idx, off, ql, PO, Pml, O, lse, st)
#define MOBA_F32_D(T, D)                        \
    switch (c.nt) {                             \
        case 1: MOBA_F32(T, D, 1);              \
        case 2: MOBA_F32(T, D, 2);              \
        case 3: MOBA_F32(T, D, 3);              \
        case 4: MOBA_F32(T, D, 4);              \
    }                                           \
    return hipErrorInvalidValue
    if (s.dtype == MOBA_F32) {
        if (s.D == 64) { MOBA_F32_D(float, 64); } else { MOBA_F32_D(float, 128); }
    } else {
        if (s.D == 64) { MOBA_F32_D(bf16_t, 64); } else { MOBA_F32_D(bf16_t, 128); }
    }
#undef MOBA_F32_D
#undef MOBA_F32
}

// ws as laid out above; the pairs (lse log2 e, -D) must be there (MOBA_BWD_PREPROCESS)
hipError_t launch_backward_f32_km(const Dims& s, const void* Q, const void* K, const void* V, const void* dO,
                                  const int32_t* idx, const int32_t* off, const int32_t* ql, void* dQ, void* dK,
                                  void* dV, void* ws, uint32_t parts, hipStream_t st)
{
    const Cut c = bwd_cut(s);
    char* p = static_cast<char*>(ws);
    const float2* ld = reinterpret_cast<const float2*>(p + backward_f32_km_ld_offset(s));
    float* PdQ = reinterpret_cast<float*>(p + bwd_partials_offset(s));
    float* sums = sums_needed(s, bwd_shares(s)) ? reinterpret_cast<float*>(p + bwd_sums_offset(s)) : nullptr;
#define MOBA_F32(T, D, NT) return bwd_launch_nt<T, D, NT>(s, c, Q, K, V, dO, ld, idx, off, ql, PdQ, sums, dQ, dK, dV, parts, st)
#define MOBA_F32_64(T)                          \
    switch (c.nt) {                             \
        case 1: MOBA_F32(T, 64, 1);             \
        case 2: MOBA_F32(T, 64, 2);             \
        case 3: MOBA_F32(T, 64, 3);             \
        case 4: MOBA_F32(T, 64, 4);             \
    }                                           \
    return hipErrorInvalidValue
#define MOBA_F32_128(T)                         \
    switch (c.nt) {                             \
        case 1: MOBA_F32(T, 128, 1);            \
        case 2: MOBA_F32(T, 128, 2);            \
        case 4: MOBA_F32(T, 128, 4);            \
    }                                           \
    return hipErrorInvalidValue
    if (s.dtype == MOBA_F32) {
        if (s.D == 64) { MOBA_F32_64(float); } else { MOBA_F32_128(float); }
    } else {
        if (s.D == 64) { MOBA_F32_64(bf16_t); } else { MOBA_F32_128(bf16_t); }
    }
#undef MOBA_F32_128
#undef MOBA_F32_64
#undef MOBA_F32
}

}  // namespace moba
