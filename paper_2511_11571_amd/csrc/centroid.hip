// Key convolution (paper Appendix B) fused with the block centroids (Section 2;
// Appendix C.1, centroid algorithm).  One pass over K: a group of D/8 lanes walks a run of
// consecutive rows of one key block top to bottom, 8 channels per lane, keeps the W-1 previous
// rows in registers for the causal depthwise filter, writes the convolved key rounded to the
// I/O type, and sums those rounded rows.  A block is cut into RS such runs (lane groups next to
// each other in one wave, so that long blocks do not leave the chip idle); their sums are added
// by shuffles in a fixed order.
//
// Bound by memory, 4 to 7 TB/s of K read (and written) where there is enough of it; short sequences by the round trips
// of a run, so eight or sixteen rows are requested together, and by the address arithmetic before the first of
// them (divisions of 64 bits took 500 instructions).  Four rows at a time, 64-bit block numbers -> now, K out of the
// caches: 16 slices of N = 8192, d = 64, B = 128: 15.6 -> 5.8 us; 32 of 16384, B = 64: 17.9 -> 14.0;
// 4 of 16384, d = 128, W = 4: 21.1 -> 15.1; 16 of 131072, d = 128, W = 4: 250 -> 225; 32 of 524288, d = 64: 385, as before.
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

template <typename T, int D, int W>
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
    if constexpr (W == 0 && sizeof(T) == 2) { MOBA_ROWS(16) }
    MOBA_ROWS(8)
    MOBA_ROWS(4)
    MOBA_ROWS(1)
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
    dim3 grid((unsigned)((runs + bpw - 1) / bpw)), block(256);
#define MOBA_CASE(WV)                                                                      \
    case WV:                                                                               \
        hipLaunchKernelGGL((centroid_kernel<T, D, WV>), grid, block, 0, st, (const T*)K, w, \
                           (T*)Keff, cent, s.heads, s.N, s.B, s.n, (uint32_t)runs, rs_log2); \
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
