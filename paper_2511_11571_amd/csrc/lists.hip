// Key-block-major query lists from query-major routing (paper Appendix C.1,
// "Reformatting Indices to Varlen Key-Block-Major").  The paper scatters with global
// atomics, which leaves the order inside a list to chance; here the lists come out
// ascending and bit-reproducible:
//   1. count: a workgroup takes a chunk of 256 consecutive queries (several, where routing is sparse) and ORs one bit per
//      (query, kept block) into an LDS bit matrix [block][256 bits]; the population
//      count of a row is the number of queries of this chunk that kept that block.
//   2. scan: per key block an exclusive scan over chunks (start of each chunk's segment
//      inside the block's list), then an exclusive scan of the block totals (blk_off).
//   3. fill: the bit matrix is rebuilt and its rows are written out in ascending order at
//      blk_off[j] + chunk start, eight lanes per row (or entry by entry, see below).
// The bit matrix lives in LDS only and covers 512 or 1024 key blocks at a time.
// Lists with places (see below) of slices with few counts take no scans: the fill pass adds the counts up itself
// (starts_from_counts(), fill_adds_up()).  Short slices take one launch instead (lists_small_kernel).
//
// A list entry holds the query in its low 24 bits (sequences are at most 2^24 long).  Where the
// key-block-major attention kernels will run (lists_with_places() of the shape and its flags) the
// high byte holds the position e of the block in the query's row of kept blocks: those kernels
// file the partial result of (query, block) under (query, e) and would otherwise have to search
// the row for the block (10-15 % of their time); elsewhere it is zero.  The fill pass gets e by walking the
// routing rows a second time: entry e of row r names block b, whose place in b's run of this
// workgroup is the number of set bits below r in b's row of the bit matrix, and is stored there at once.
// (Collecting e per run in LDS first and writing row by row took longer at every shape measured; without
// places the walk over the rows of the matrix is the faster one up to 4096 blocks.)
// us, both passes and scans, before -> after: 32 slices, N = 524288, 4096 blocks, k = 8: 4180 -> 2890
// (with several chunks to a workgroup since: 1935); 16 slices, N = 131072, 1024 blocks, k = 8: 261 -> 151, 2048 blocks, k = 32: 693 -> 637; 8 slices, N = 131072,
// 4096 blocks, k = 32: 552 -> 356; 16 slices, N = 16384, 256 blocks, k = 16: 55 -> 38.  Bound by the scattered
// 4-byte stores and, in the count, by the walk over a matrix that is mostly empty.
#include <algorithm>

#include "mfma.h"

namespace moba {

constexpr int kRangeMax = 1024;                 // key blocks per LDS bit matrix at most (32 KB)
constexpr int kRangeLong = 512;                 // the shorter one, see launch_build_lists
constexpr int kListQ = kChunkQ;                  // queries per workgroup: one chunk
constexpr int kWords = kListQ / 32;             // 8 words of 32 query bits per block
constexpr int kQueryBits = 24;                  // low bits of a list entry: the query

// f(r, b, e) for every entry b = row r's e-th of the routing rows r = 0 .. rows-1 of this workgroup
// (k entries per row, rows contiguous in memory), all NT threads, 16-byte loads when the row length
// allows.  The row and place of a thread's entries advance by additions (one division per thread).
template <int NT = 256, typename F>
__device__ __forceinline__ void for_each_entry_slot(const int32_t* __restrict__ rows0, int rows, int k,
                                                    int tid, F f)
{
    const int total = rows * k;
    if ((k & 3) == 0) {
        const int4* p4 = reinterpret_cast<const int4*>(rows0);
        const int n4 = total >> 2;
        const int dr = 4 * NT / k, de = 4 * NT % k;         // NT pieces of four entries further on
        int r = 4 * tid / k, e = 4 * tid - r * k;           // a 16-byte piece never straddles rows
        for (int i0 = tid; i0 < n4; i0 += 4 * NT) {
            int4 v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u)
                v[u] = i0 + u * NT < n4 ? p4[i0 + u * NT] : make_int4(-1, -1, -1, -1);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                f(r, v[u].x, e); f(r, v[u].y, e + 1); f(r, v[u].z, e + 2); f(r, v[u].w, e + 3);
                r += dr;
                e += de;
                if (e >= k) { e -= k; ++r; }
            }
        }
    } else {
        const int dr = NT / k, de = NT % k;
        int r = tid / k, e = tid - r * k;
        for (int i = tid; i < total; i += NT) {
            f(r, rows0[i], e);
            r += dr;
            e += de;
            if (e >= k) { e -= k; ++r; }
        }
    }
}

// the same without the place: f(r, b)
template <typename F>
__device__ __forceinline__ void for_each_entry(const int32_t* __restrict__ rows0, int rows, int k, int tid, F f)
{
    for_each_entry_slot(rows0, rows, k, tid, [&](int r, int b, int) { f(r, b); });
}

// sum of `mine` over the threads before this one (256 threads, one barrier)
__device__ __forceinline__ int sum_before(int mine, int* wsum, int tid)
{
    int incl = mine;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const int up = __shfl_up(incl, o, kWave);
        if (tid % kWave >= o) incl += up;
    }
    if (tid % kWave == kWave - 1) wsum[tid / kWave] = incl;
    __syncthreads();
    int before = incl - mine;
    for (int w = 0; w < tid / kWave; ++w) before += wsum[w];
    return before;
}

// What lists_scan_kernel and lists_offsets_kernel leave, worked out by the fill pass itself from the counts of all
// chunks: start[j] of chunk c for the n <= kRange blocks; the last chunk's workgroup writes off[0 .. n].
// scratch: 2 * kRange words
template <int kRange>
__device__ __forceinline__ void starts_from_counts(const int32_t* __restrict__ counts, int32_t* __restrict__ off, int n,
                                                   int nchunk, int c, int32_t* scratch, int32_t* start, int tid)
{
    constexpr int EPT = kRange / 256;
    __shared__ int wsum[4];
    int32_t* total = scratch;
    int32_t* before = scratch + kRange;
    for (int j = tid; j < n; j += 256) total[j] = before[j] = 0;
    __syncthreads();
    const int dc = 256 / n, dj = 256 - dc * n;               // 256 counts further on
    int ch = tid / n, j = tid - ch * n;
#pragma unroll 4
    for (int i = tid; i < nchunk * n; i += 256) {
        const int v = counts[i];
        if (v) {
            atomicAdd(&total[j], v);
            if (ch < c) atomicAdd(&before[j], v);
        }
        ch += dc;
        j += dj;
        if (j >= n) { j -= n; ++ch; }
    }
    __syncthreads();
    int v[EPT], sum = 0;
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
        v[e] = tid * EPT + e < n ? total[tid * EPT + e] : 0;
        sum += v[e];
    }
    int run = sum_before(sum, wsum, tid);
    const bool last = c == nchunk - 1;
    if (last && tid == 0) off[0] = 0;
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
        const int b = tid * EPT + e;
        if (b >= n) break;
        start[b] = run + before[b];
        run += v[e];
        if (last) off[b + 1] = run;
    }
    __syncthreads();
}

// kRange: key blocks per LDS bit matrix (blockIdx.y counts the ranges of a slice's blocks).
// A workgroup takes `group` chunks one after the other; the counts are those of all of them, and `groups` of a slice are scanned.
// SELF (fill, one range, one chunk): no scans went before, see above
template <bool FILL, bool SLOTS, int kRange, bool SELF = false>
__global__ __launch_bounds__(256) void lists_chunk_kernel(
    const int32_t* __restrict__ idx, int32_t* __restrict__ cnt2, int32_t* __restrict__ off,
    int32_t* __restrict__ ql, int N, int B, int n, int k, int groups, int group, int64_t R, int bh)
{
    __shared__ __align__(16) uint32_t mask[kRange * kWords];
    __shared__ int32_t start[FILL ? kRange : 1];         // where the next chunk's queries start in each list
    // consecutive query chunks of a slice go to the same XCD: the 128-byte lines of a block's
    // list are completed by neighbouring chunks and should meet in one L2 before they are written back
    int c, s;
    if (!schedule(blockIdx.x, bh, groups, s, c)) return;
    const int lo = blockIdx.y * kRange;
    const int hi = min(n, lo + kRange);
    const int first = c * group * kListQ, end = min(N, first + group * kListQ);
    // kept blocks are < own block of the query: of a chunk's last, of the last of all
    auto blocks = [&](int queries_end) { return min(hi, (queries_end - 1) / B) - lo; };
    const int most = blocks(end);
    const int tid = threadIdx.x;
    int32_t* crow = cnt2 + ((int64_t)s * (groups + 1) + c) * n + lo;
    if constexpr (SELF)
        starts_from_counts<kRange>(cnt2 + (int64_t)s * (groups + 1) * n, off + (int64_t)s * (n + 1), n, groups, c,
                                   reinterpret_cast<int32_t*>(mask), start, tid);
    if (most <= 0) {
        if (!FILL)
            for (int j = tid; j < hi - lo; j += 256) crow[j] = 0;
        return;
    }
    for (int i = tid; i < most * kWords; i += 256) mask[i] = 0u;
    if (FILL && !SELF) {
        const int32_t* orow = off + (int64_t)s * (n + 1) + lo;
        for (int j = tid; j < most; j += 256) {
            start[j] = orow[j] + crow[j];
        }
    }
    auto bits_of = [&](int j) {
        int c0 = 0;
#pragma unroll
        for (int wd = 0; wd < kWords; ++wd) c0 += __popc(mask[j * kWords + wd]);
        return c0;
    };
    auto clear = [&](int j) {
#pragma unroll
        for (int wd = 0; wd < kWords; ++wd) mask[j * kWords + wd] = 0u;
    };
    int count[FILL ? 1 : kRange / 256] = {};             // of blocks tid + 256 u
    for (int t0 = first; t0 < end; t0 += kListQ) {
        const int rows = min(end - t0, kListQ), nblk = blocks(t0 + rows);
        if (nblk <= 0) continue;
        const bool more = t0 + kListQ < end;
        __syncthreads();
        const int32_t* rows0 = idx + ((int64_t)s * N + t0) * k;
        // only past blocks count: lists never exceed R
        for_each_entry(rows0, rows, k, tid, [&](int r, int b) {
            b -= lo;
            // (block b + lo lies before the own block of query t0 + r: its last key does)
            if (b >= 0 && b < nblk && (b + lo + 1) * B <= t0 + r) atomicOr(&mask[b * kWords + (r >> 5)], 1u << (r & 31));
        });
        __syncthreads();
        if constexpr (!FILL) {
#pragma unroll
            for (int u = 0; u < kRange / 256; ++u) {
                const int j = tid + 256 * u;
                if (j >= nblk) break;
                count[u] += bits_of(j);
                if (more) clear(j);
            }
        } else if constexpr (SLOTS) {
            int32_t* qs = ql + (int64_t)s * R;
            for_each_entry_slot(rows0, rows, k, tid, [&](int r, int b, int e) {
                b -= lo;
                if (b >= 0 && b < nblk && (b + lo + 1) * B <= t0 + r) {
                    const uint32_t* mrow = mask + b * kWords;
                    const int last = r >> 5;
                    int rank = 0;
#pragma unroll
                    for (int wd = 0; wd < kWords; ++wd) {
                        const uint32_t below = wd < last ? ~0u : wd == last ? (1u << (r & 31)) - 1u : 0u;
                        rank += __popc(mrow[wd] & below);
                    }
                    const int64_t pos = (int64_t)start[b] + rank;
                    // a routing that breaks the contract (repeats, too many kept blocks) must not
                    // write outside the slice's lists
                    if (pos < R) qs[pos] = (t0 + r) | e << kQueryBits;
                }
            });
            if (more) {
                __syncthreads();
                for (int j = tid; j < nblk; j += 256) {
                    start[j] += bits_of(j);
                    clear(j);
                }
            }
        } else {
            // Eight lanes per block, one 32-query word each: a lane writes the queries of its word
            // after those of the lanes before it.  The 256 queries of a chunk are neighbours
            // in every list, so a store instruction touches one short run of addresses per block.
            int32_t* qs = ql + (int64_t)s * R;
            const int lane8 = tid & 7;
            for (int b = tid >> 3; b < nblk; b += 256 / 8) {
                uint32_t word = mask[b * kWords + lane8];
                const int cnt = __popc(word);
                int incl = cnt;
#pragma unroll
                for (int o = 1; o < 8; o <<= 1) {
                    const int up = __shfl_up(incl, o, 8);
                    if (lane8 >= o) incl += up;
                }
                const int at = start[b];
                int64_t pos = (int64_t)at + (incl - cnt);
                while (word) {
                    if (pos < R) qs[pos] = t0 + 32 * lane8 + (__ffs(word) - 1);      // (as above)
                    ++pos;
                    word &= word - 1u;
                }
                if (more) {                              // (the eight lanes of a block are one wave's: all have read)
                    mask[b * kWords + lane8] = 0u;
                    if (lane8 == 7) start[b] = at + incl;
                }
            }
        }
    }
    if constexpr (!FILL) {
#pragma unroll
        for (int u = 0; u < kRange / 256; ++u)
            if (tid + 256 * u < hi - lo) crow[tid + 256 * u] = count[u];
    }
}

// per slice and key block: cnt2[c][j] <- sum_{c' < c} cnt2[c'][j] (row nchunk: the total).
// A workgroup takes 32 key blocks; 8 threads per block share the chunks, kScanAhead counts read before the first of
// them is used (one at a time, each waits for the store before it: 32 slices of 2048 chunks x 4096 blocks
// 777 -> 740 us, three passes over memory; 16 of 512 x 2048 51 -> 31; 32 of 256 x 512 17.3 -> 9.7).
constexpr int kScanAhead = 8;

__global__ __launch_bounds__(256) void lists_scan_kernel(int32_t* __restrict__ cnt2,
                                                         int32_t* __restrict__ off, int n,
                                                         int nchunk)
{
    __shared__ int part[8][33];
    const int s = blockIdx.y, tid = threadIdx.x;
    const int jj = tid & 31, seg = tid >> 5;
    const int j = blockIdx.x * 32 + jj;
    int32_t* cs = cnt2 + (int64_t)s * (nchunk + 1) * n;
    const int per = (nchunk + 7) / 8;
    const int c0 = min(nchunk, seg * per), c1 = min(nchunk, c0 + per);
    int sum = 0;
    if (j < n)
        for (int c = c0; c < c1; c += kScanAhead) {
            int v[kScanAhead];
#pragma unroll
            for (int u = 0; u < kScanAhead; ++u) v[u] = c + u < c1 ? cs[(int64_t)(c + u) * n + j] : 0;
#pragma unroll
            for (int u = 0; u < kScanAhead; ++u) sum += v[u];
        }
    part[seg][jj] = sum;
    __syncthreads();
    int run = 0, total = 0;
#pragma unroll
    for (int g = 0; g < 8; ++g) {
        const int v = part[g][jj];
        if (g < seg) run += v;
        total += v;
    }
    if (j < n) {
        for (int c = c0; c < c1; c += kScanAhead) {
            int v[kScanAhead];
#pragma unroll
            for (int u = 0; u < kScanAhead; ++u) v[u] = c + u < c1 ? cs[(int64_t)(c + u) * n + j] : 0;
#pragma unroll
            for (int u = 0; u < kScanAhead; ++u) {
                if (c + u < c1) cs[(int64_t)(c + u) * n + j] = run;
                run += v[u];
            }
        }
        if (seg == 0) {
            cs[(int64_t)nchunk * n + j] = total;
            off[(int64_t)s * (n + 1) + j + 1] = total;
        }
    }
}

// per slice: off[j] <- sum_{j' < j} total[j'] (off[j + 1] holds total[j] on entry)
__global__ __launch_bounds__(256) void lists_offsets_kernel(int32_t* __restrict__ off, int n)
{
    __shared__ int wsum[4];
    const int s = blockIdx.x, tid = threadIdx.x;
    int32_t* os = off + (int64_t)s * (n + 1);
    const int seg = (n + 255) / 256;
    const int a = min(n, tid * seg), b = min(n, a + seg);
    int sum = 0;
    for (int j = a; j < b; ++j) sum += os[j + 1];
    int run = sum_before(sum, wsum, tid);
    if (tid == 0) os[0] = 0;
    for (int j = a; j < b; ++j) { run += os[j + 1]; os[j + 1] = run; }
}

// ---- short slices: one launch.  A workgroup holds the bit matrix of the slice's blocks up to the last of
// its `own` blocks, from all queries, and writes the lists of its blocks: the words of their rows, one row
// after the other, are in list order, so one scan over the threads gives every word its place; the bits of
// the rows before them are where the first list starts.  Every workgroup of a slice walks the slice's whole
// routing (from its L2), which buys the three launches and the counts in memory that lists_chunk_kernel and
// its scans need.  Bound by that walk: an LDS atomic per entry in every workgroup.
// us, four launches -> one: 2 slices, N = 2048, k = 3: 19 -> 9; 8 slices, N = 4096, k = 7: 25 -> 17;
// 16 slices, N = 8192, k = 8: 27 -> 26 (65536 entries per slice, no longer taken).
constexpr int kSmallThreads = 1024;
constexpr size_t kSmallLds = 144 << 10;         // bit matrix and places, of the 160 KB of a compute unit
constexpr int kSmallEntries = 1 << 15;          // routing entries per slice

struct SmallLists {
    int own, wgs;                               // key blocks per workgroup, workgroups per slice
    size_t lds;
    bool ok;
};
__host__ __device__ inline int small_row_words(int N) { return (N + 31) / 32 | 1; }   // (odd: rows on different banks)

template <bool SLOTS>
__global__ __launch_bounds__(kSmallThreads) void lists_small_kernel(
    const int32_t* __restrict__ idx, int32_t* __restrict__ off, int32_t* __restrict__ ql, int N, int B, int n, int k,
    int own, int wgs, int64_t R, int bh)
{
    extern __shared__ __align__(16) uint32_t mask[];     // [hi][words], then SLOTS: e of (own block, query), bytes
    __shared__ int sums[2][kSmallThreads / kWave];
    int s, c;
    if (!schedule(blockIdx.x, bh, wgs, s, c)) return;
    const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
    const int words = small_row_words(N);
    const int lo = c * own, hi = min(n, lo + own);
    uint8_t* slot = reinterpret_cast<uint8_t*>(mask + (size_t)min(n, wgs * own) * words);
    for (int i = tid; i < hi * words; i += kSmallThreads) mask[i] = 0u;
    __syncthreads();
    // only past blocks count: lists never exceed R
    for_each_entry_slot<kSmallThreads>(idx + (int64_t)s * N * k, N, k, tid, [&](int r, int b, int e) {
        if (b < 0 || b >= hi || (b + 1) * B > r) return;
        atomicOr(&mask[b * words + (r >> 5)], 1u << (r & 31));
        if (SLOTS && b >= lo) slot[(b - lo) * N + r] = (uint8_t)e;
    });
    __syncthreads();
    int before = 0;                                      // entries of the blocks before lo
    for (int i = tid; i < lo * words; i += kSmallThreads) before += __popc(mask[i]);
    const int mywords = (hi - lo) * words, per = (mywords + kSmallThreads - 1) / kSmallThreads;
    const uint32_t* mine = mask + lo * words;
    const int a = min(mywords, tid * per), z = min(mywords, a + per);
    int count = 0;
    for (int i = a; i < z; ++i) count += __popc(mine[i]);
    int incl = count;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const int up = __shfl_up(incl, o, kWave);
        before += __shfl_xor(before, o, kWave);
        if (lane >= o) incl += up;
    }
    if (lane == kWave - 1) {
        sums[0][wave] = incl;
        sums[1][wave] = before;
    }
    __syncthreads();
    int pos = incl - count;
    for (int w = 0; w < kSmallThreads / kWave; ++w) pos += sums[1][w] + (w < wave ? sums[0][w] : 0);
    int32_t* os = off + (int64_t)s * (n + 1);
    int32_t* qs = ql + (int64_t)s * R;
    int b = a / words, w = a - b * words;
    for (int i = a; i < z; ++i) {
        if (w == 0) os[lo + b] = pos;
        uint32_t word = mine[i];
        while (word) {
            const int r = 32 * w + (__ffs(word) - 1);
            // a routing that breaks the contract must not write outside the slice's lists
            if (pos < R) qs[pos] = SLOTS ? r | (int)slot[b * N + r] << kQueryBits : r;
            ++pos;
            word &= word - 1u;
        }
        if (++w == words) { w = 0; ++b; }
    }
    if (hi == n && z == mywords && a < z) os[n] = pos;
}

// Blocks per workgroup: as few as keep the launch within one workgroup per compute unit.  The line is set by
// the walk (see above: half the entries of the shape that gains nothing) and by what the LDS holds.
static SmallLists small_lists(const Dims& s)
{
    SmallLists p = {0, 0, 0, false};
    if (s.k <= 0 || s.R <= 0 || s.k > 255) return p;
    p.own = (int)(((int64_t)s.n * s.bh + 255) / 256);
    p.wgs = (s.n + p.own - 1) / p.own;
    const size_t bits = sizeof(uint32_t) * (size_t)s.n * small_row_words(s.N);
    p.lds = bits + (lists_with_places(s) ? (size_t)p.own * s.N : 0);
    p.ok = p.lds <= kSmallLds && (int64_t)s.N * s.k <= kSmallEntries;
    return p;
}

template <bool SLOTS>
static hipError_t small_launch(const Dims& s, const SmallLists& p, const int32_t* idx, int32_t* off, int32_t* ql,
                               hipStream_t st)
{
    hipError_t e = ensure_dynamic_lds((const void*)lists_small_kernel<SLOTS>, p.lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((lists_small_kernel<SLOTS>), dim3((unsigned)schedule_grid(s.bh, p.wgs)), dim3(kSmallThreads), p.lds,
                       st, idx, off, ql, s.N, s.B, s.n, s.k, p.own, p.wgs, s.R, s.bh);
    return hipGetLastError();
}

// Most counts of a slice (chunks x blocks) that every workgroup of the fill pass adds up for itself, in place of
// two launches, and most such additions of all workgroups together: a workgroup's own are a few rounds of loads and LDS
// adds before its work, all workgroups' are time of the chip that two scans do not take.
// us of the whole builder, scans -> itself, by counts / workgroups:
//   2048 / 512 (16 slices, N = 8192, 64 blocks) 17.1 -> 13.6;  4096 / 64 16.6 -> 13.9;  4096 / 512 17.2 -> 14.5;
//   6144 / 768 18.7 -> 17.4;  6084 / 156 16.7 -> 16.1;  8192 / 64 17.1 -> 18.3;  9216 / 96 17.5 -> 19.6
//   (the first line: between 6144 and 8192);
//   4608 / 768 (3.5 M additions) 18.6 -> 16.6;  2048 / 3072 (6.3 M) 38.7 -> 38.8;  4608 / 1536 (7.1 M) 50.7 -> 51.5;
//   4096 / 2048 (8.4 M) 33.7 -> 33.0;  4096 / 3072 (12.6 M) 67.8 -> 68.1;  6084 / 3744 (22.8 M) 47.5 -> 54.5;
//   4096 / 6144 (25 M) 43.7 -> 52.6  (the second: at 8 M)
constexpr int kSelfCounts = 6144;
constexpr int64_t kSelfAdditions = (int64_t)8 << 20;
static bool fill_adds_up(const Dims& s)
{
    const int64_t counts = (int64_t)s.nchunk * s.n;
    return s.R > 0 && counts <= kSelfCounts && counts * s.nchunk * s.bh <= kSelfAdditions;
}

// Chunks that a workgroup takes one after the other: what they cost in memory is then one count per block, written, scanned (two
// reads and a write) and read back, for all of them.  As many as leave 4096 workgroups and bring a block about two queries: beyond
// that the lists cost more than the counts, and workgroups far apart share fewer of the lists' lines in an L2 at a time.
// us of the whole builder, one chunk -> this many: 32 slices, N = 524288, 4096 blocks, k = 8 (4 chunks) 2890 -> 1935;
// 16 slices, N = 524288, 4096 blocks, k = 2 (16) 1176 -> 421; 16 slices, N = 261888, 2728 blocks, k = 10 (2) 807 -> 689, with 4 765,
// 8 869; 64 slices, N = 65536, 2048 blocks, k = 4 (4) 290 -> 204; 16 slices, N = 131072, 2048 blocks, k = 32 (1) 637, with 4 714.
constexpr int kGroupWgs = 4096, kGroupRows = 2, kGroupMost = 16;
static int chunks_together(const Dims& s, int nranges)
{
    const int64_t wgs = (int64_t)s.bh * s.nchunk * nranges;
    const int64_t group = std::min<int64_t>(wgs / kGroupWgs, (int64_t)kGroupRows * s.n / std::max(1, kListQ * s.k));
    return (int)std::min<int64_t>(std::max<int64_t>(group, 1), kGroupMost);
}

template <int RANGE>
static hipError_t build_lists_launch(const Dims& s, const int32_t* idx, int32_t* off, int32_t* ql,
                                     int32_t* cnt2, hipStream_t st)
{
    const int nranges = (s.n + RANGE - 1) / RANGE;
    const int group = chunks_together(s, nranges), groups = (s.nchunk + group - 1) / group;
    dim3 grid(schedule_grid(s.bh, groups), nranges), block(256);
    hipLaunchKernelGGL((lists_chunk_kernel<false, false, RANGE>), grid, block, 0, st, idx, cnt2, off, ql, s.N, s.B,
                       s.n, s.k, groups, group, s.R, s.bh);
    static_assert(kKeyMajorMaxTopk <= 127, "the place of a block in the high byte of an entry");
    const bool places = lists_with_places(s);
#define MOBA_FILL(PLACES, SELF)                                                                                          \
    hipLaunchKernelGGL((lists_chunk_kernel<true, PLACES, RANGE, SELF>), grid, block, 0, st, idx, cnt2, off, ql, s.N, s.B, \
                       s.n, s.k, groups, group, s.R, s.bh)
    // (without places this range serves slices of more than kRangeMax blocks, which have too many counts)
    if constexpr (RANGE == kRangeLong) {
        if (places && s.n <= RANGE && group == 1 && fill_adds_up(s)) {
            MOBA_FILL(true, true);
            return hipGetLastError();
        }
    }
    hipLaunchKernelGGL(lists_scan_kernel, dim3((s.n + 31) / 32, s.bh), block, 0, st, cnt2, off, s.n,
                       groups);
    hipLaunchKernelGGL(lists_offsets_kernel, dim3(s.bh), block, 0, st, off, s.n);
    if (s.R > 0) {
        if (places) MOBA_FILL(true, false);
        else MOBA_FILL(false, false);
    }
#undef MOBA_FILL
    return hipGetLastError();
}

// Up to kRangeMax blocks one range covers a slice and a workgroup reads its routing rows once.
// Beyond that the rows are read once per range anyway, and without places a workgroup's cost is that of
// walking the rows of its bit matrix, however few pairs fall into it: smaller ranges, more workgroups.
// With places the rows are walked by the count alone: the full range (8 slices, N = 131072, 4096 blocks,
// k = 60: 830 us against 1080 with 512), but the short one where it covers a slice (16 slices, N = 65536,
// 512 blocks, k = 8: 68 against 72; half the LDS, more workgroups in flight).
hipError_t launch_build_lists(const Dims& s, const int32_t* idx, int32_t* off, int32_t* ql,
                              int32_t* cnt2, hipStream_t st)
{
    const SmallLists p = small_lists(s);
    if (p.ok) return lists_with_places(s) ? small_launch<true>(s, p, idx, off, ql, st) : small_launch<false>(s, p, idx, off, ql, st);
    const bool full = lists_with_places(s) ? s.n > kRangeLong : s.n <= kRangeMax;
    return full ? build_lists_launch<kRangeMax>(s, idx, off, ql, cnt2, st)
                : build_lists_launch<kRangeLong>(s, idx, off, ql, cnt2, st);
}

}  // namespace moba
