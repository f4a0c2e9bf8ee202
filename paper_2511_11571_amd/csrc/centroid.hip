// Key convolution (paper Appendix B) fused with the block centroids (Section 2;
// Appendix C.1, centroid algorithm).  One pass over K: a group of D/8 lanes walks a run of
// consecutive rows of one key block top to bottom, 8 channels per lane, keeps the W-1 previous
// rows in registers for the causal depthwise filter, writes the convolved key rounded to the
// I/O type, and sums those rounded rows.  A block is cut into RS such runs (lane groups next to
// each other in one wave, so that long blocks do not leave the chip idle); their sums are added
// by shuffles in a fixed order.
//
// Bound by memory, 4 to 7 TB/s of K read (and written) where there is enough of it; short sequences by the round trips
// of a run, so several rows are requested together (rows_together()), and by the address arithmetic before the first
// of them (divisions of 64 bits took 500 instructions).  Four rows at a time, 64-bit block numbers -> now, K out of the
// caches: 16 slices of N = 8192, d = 64, B = 128: 15.4 -> 5.4 us; 32 of 16384, B = 64: 16.5 -> 13.2;
// 4 of 16384, d = 128, W = 4: 20.7 -> 15.1; 16 of 131072, d = 128, W = 4: 240 -> 217; 32 of 524288, d = 64: 370 -> 371.
// (Right after a backward whose dQ merge streams its partials the call takes longer: 406 us at the last of these, see MergeRow.)
#include "common.h"

namespace moba {

// U rows of a run: all of them are on their way before the first is used
template <typename T, int D, int W, int U>
__device__ __forceinline__ void centroid_rows(const T* __restrict__ src, T* __restrict__ dst, bool store,
                                              const float (&wr)[W > 0 ? W : 1][8], float (&win)[W > 1 ? W - 1 : 1][8],
                                              float (&acc)[8])
{
    typename Vec8<T>::Raw raw[U];
#pragma unroll
    for (int u = 0; u < U; ++u) raw[u] = Vec8<T>::raw(src + u * D);
    if constexpr (W == 0) {
        if (store)
#pragma unroll
            for (int u = 0; u < U; ++u) *reinterpret_cast<typename Vec8<T>::Raw*>(dst + u * D) = raw[u];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        float x[8], y[8];
        Vec8<T>::unpack(raw[u], x);
        if constexpr (W > 0) {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                float a = wr[0][e] * x[e];
#pragma unroll
                for (int l = 1; l < W; ++l) a = fmaf(wr[l][e], win[l - 1][e], a);
                y[e] = x[e] + a * __builtin_amdgcn_rcpf(1.f + __expf(-a));     // SiLU; sigmoid to ~1 ulp
            }
#pragma unroll
            for (int l = W - 1; l > 1; --l)
#pragma unroll
                for (int e = 0; e < 8; ++e) win[l - 1][e] = win[l - 2][e];
            if constexpr (W > 1) {
#pragma unroll
                for (int e = 0; e < 8; ++e) win[0][e] = x[e];
            }
            Vec8<T>::store(dst + u * D, y);
#pragma unroll
            for (int e = 0; e < 8; ++e) acc[e] += Vec8<T>::round(y[e]);
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) acc[e] += x[e];
        }
    }
}

// MOST: rows of a run that are requested together at most (1: the compiler's unrolling by four)
template <typename T, int D, int W, int MOST>
__global__ __launch_bounds__(256) void centroid_kernel(
    const T* __restrict__ K, const float* __restrict__ w, T* __restrict__ Keff,
    float* __restrict__ cent, int heads, int N, int B, int n, uint32_t total_runs, int rs_log2)
{
    constexpr int G = D / 8;          // lanes per run of rows
    constexpr int BPW = 256 / G;      // runs per workgroup (a multiple of RS)
    constexpr int WW = W > 1 ? W - 1 : 1;
    // (a launch has fewer than 2^32 threads, D/8 of them for a run: 32 bits hold the runs)
    const uint32_t run = blockIdx.x * BPW + threadIdx.x / G;
    const bool live = run < total_runs;                     // (idle lanes still take part in the shuffles)
    const uint32_t blk = live ? run >> rs_log2 : 0u;
    const int RS = 1 << rs_log2, sp = live ? (int)(run & (RS - 1)) : 0;
    const int CH = B >> rs_log2;                            // rows per run
    const uint32_t s = blk / (uint32_t)n;
    const int j = (int)(blk - s * (uint32_t)n);
    const int first = j * B + sp * CH;                      // first row of the run inside the slice
    const int64_t row0 = (int64_t)s * N + first;
    const int part = threadIdx.x % G;
    const T* src = K + row0 * D + part * 8;
    T* dst = Keff + row0 * D + part * 8;
    const bool store = Keff != nullptr;                     // (always, where there is a filter)

    float wr[W > 0 ? W : 1][8];
    float win[WW][8];                  // win[l-1] = row t-l
    if constexpr (W > 0) {
        const float* wh = w + ((int64_t)(s % (uint32_t)heads) * D + part * 8) * W;
#pragma unroll
        for (int e = 0; e < 8; ++e)
#pragma unroll
            for (int l = 0; l < W; ++l) wr[l][e] = wh[e * W + l];
#pragma unroll
        for (int l = 1; l < W; ++l) {
            if (first - l >= 0) Vec8<T>::load(src - (int64_t)l * D, win[l - 1]);
            else {
#pragma unroll
                for (int e = 0; e < 8; ++e) win[l - 1][e] = 0.f;
            }
        }
    }

    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    int left = live ? CH : 0;
#define MOBA_ROWS(U) \
    for (; left >= U; left -= U, src += U * D, dst += U * D) centroid_rows<T, D, W, U>(src, dst, store, wr, win, acc);
    if constexpr (MOST == 1) {
#pragma unroll 4
        MOBA_ROWS(1)
    } else {
        if constexpr (MOST >= 16) { MOBA_ROWS(16) }
        if constexpr (MOST >= 8) { MOBA_ROWS(8) }
        MOBA_ROWS(4)
        MOBA_ROWS(1)
    }
#undef MOBA_ROWS
    for (int o = G; o < G * RS; o <<= 1)
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] += __shfl_xor(acc[e], o, kWave);
    if (live && sp == 0) {
        float out[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) out[e] = acc[e] / (float)B;
        Vec8<float>::store(cent + (int64_t)blk * D + part * 8, out);
    }
}

// Rows requested together.
// bf16 without a filter: 16, but 8 where a run has just 16 rows of 128 bytes and the chip's lanes (2^19) are all taken:
// waves of 86 registers, five to a SIMD, are then worth less than eight of 54.  With a filter: 8 (150 registers; 16: 214).
// fp32 (a lane's two 16-byte loads of a row share its lines, and beyond 32 KB in flight a compute unit may have lost
// them before the second): 16 in runs of 16 (d = 64; 128: 17) to 32 rows, but with a filter at d = 128 no more than 8, and
// 4 with two lags where a wave on every SIMD walks long runs; 8 otherwise, and one after the other in the short runs of
// a call that takes all lanes without a filter.  A filter of one lag (few instructions between the loads): one after
// the other.
// us with 1 / 4 / 8 / 16 rows, slices x N:
//   bf16  d = 64, B = 128, 32 x 512 K 368 / 369 / 371 / 379, 32 x 32 K 26.2 / 24.8 / 25.1 / 25.6, 16 x 8 K - / 6.2 / 5.8 / 5.4;
//         B = 512, 32 x 128 K - / 96 / 117 / 111;  d = 128, B = 64, 16 x 32 K - / 29.8 / 31.0 / 26.2
//         W = 4, 32 x 64 K, d = 64, B = 64 133 / 112 / 117 / 141, 16 x 8 K, d = 128, B = 128 36 / 24.7 / 23.7 / 23.0
//   fp32  d = 64, 32 x 64 K, B = 64 92 / 94 / 97 / 97, B = 128 97 / 98 / 100 / 90, B = 256 114 / 121 / 112 / 107;
//         d = 128, 32 x 64 K, B = 128 190 / 200 / 200 / 180; 16 x 8 K, B = 64 15.4 / 16.0 / 13.2 / 13.9
//         W = 1, d = 64, B = 256, 32 x 64 K 227 / 286 / 299 / 276;  W = 3, d = 64, B = 256 262 / 281 / 240 / 216;
//         W = 2, d = 128, B = 128, 16 x 8 K 31.6 / 30.4 / 34.0 / 36.3, 8 x 8 K 27.4 / 22.0 / 19.6 / 23.2, B = 256,
//         32 x 32 K 212 / 209 / 224 / 281;  W = 3, 32 x 32 K 229 / 237 / 228 / 252;  W = 8, d = 64, B = 64, 32 x 64 K 219 / 229 / 225 / 303
template <typename T, int D>
static int rows_together(int W, int run_rows, int64_t lanes)
{
    const bool full = lanes >= (int64_t)1 << 19;
    if (sizeof(T) == 2) return W > 0 || (D == 64 && run_rows == 16 && full) ? 8 : 16;
    if (W == 1) return 1;
    if (W > 4) return 8;
    if (D == 128 && W > 0) return W == 2 && run_rows > 16 && lanes >= (int64_t)1 << 16 ? 4 : 8;
    if (run_rows >= (D == 64 ? 16 : 17) && run_rows <= 32) return 16;
    return D == 64 && W == 0 && run_rows < 16 && full ? 1 : 8;
}

template <typename T, int D, int W>
static void launch_rows(int most, dim3 grid, hipStream_t st, const Dims& s, const T* K, const float* w, T* Keff,
                        float* cent, uint32_t runs, int rs_log2)
{
    constexpr bool F = sizeof(T) == 4;                     // (what rows_together() can say is compiled, nothing else)
#define MOBA_LAUNCH(COUNT)                                                                                          \
    {                                                                                                               \
        hipLaunchKernelGGL((centroid_kernel<T, D, W, COUNT>), grid, dim3(256), 0, st, K, w, Keff, cent, s.heads, s.N, \
                           s.B, s.n, runs, rs_log2);                                                                \
        return;                                                                                                     \
    }
    if constexpr (F && (W == 1 || (W == 0 && D == 64))) { if (most == 1) MOBA_LAUNCH(1) }
    if constexpr (F && D == 128 && W == 2) { if (most == 4) MOBA_LAUNCH(4) }
    if constexpr (F ? W == 0 || (D == 64 && W >= 2 && W <= 4) : W == 0) { if (most == 16) MOBA_LAUNCH(16) }
    if constexpr (F ? W != 1 : W > 0 || D == 64) MOBA_LAUNCH(8)
#undef MOBA_LAUNCH
}

template <typename T, int D>
static hipError_t launch_w(const Dims& s, const void* K, const float* w, void* Keff, float* cent,
                           hipStream_t st)
{
    const int64_t total = (int64_t)s.bh * s.n;
    const int bpw = 256 / (D / 8);
    // runs per block: as many as fit a wave side by side, of at least 8 rows each
    int rs_log2 = 0;
    while ((2 << rs_log2) * (D / 8) <= kWave && s.B % (2 << rs_log2) == 0 && s.B / (2 << rs_log2) >= 8) ++rs_log2;
    const int64_t runs = total << rs_log2;
    const dim3 grid((unsigned)((runs + bpw - 1) / bpw));
    const int most = rows_together<T, D>(s.W, s.B >> rs_log2, runs * (D / 8));
#define MOBA_CASE(WV)                                                                                        \
    case WV:                                                                                                 \
        launch_rows<T, D, WV>(most, grid, st, s, (const T*)K, w, (T*)Keff, cent, (uint32_t)runs, rs_log2); \
        break;
    switch (s.W) {
        MOBA_CASE(0) MOBA_CASE(1) MOBA_CASE(2) MOBA_CASE(3) MOBA_CASE(4)
        MOBA_CASE(5) MOBA_CASE(6) MOBA_CASE(7) MOBA_CASE(8)
        default: return hipErrorInvalidValue;
    }
#undef MOBA_CASE
    return hipGetLastError();
}

hipError_t launch_centroids(const Dims& s, const void* K, const float* w, void* Keff, float* cent,
                            hipStream_t st)
{
    if (s.dtype == MOBA_BF16)
        return s.D == 64 ? launch_w<bf16_t, 64>(s, K, w, Keff, cent, st)
                         : launch_w<bf16_t, 128>(s, K, w, Keff, cent, st);
    return s.D == 64 ? launch_w<float, 64>(s, K, w, Keff, cent, st)
                     : launch_w<float, 128>(s, K, w, Keff, cent, st);
}

}  // namespace moba
