// MoBA forward, key-block major, for sparse routing (paper Section 4.2, forward pass with
// gather-and-densify: one logical key block at a time, the queries routed to it gathered into
// dense tiles).  The query-tile kernel of attn_fwd_mfma.hip needs a 256-query tile to meet a key
// block with many of its rows; with few kept blocks out of very many (long sequences) a tile
// meets a block with one or two rows and the work per (query, block) pair explodes.  Here a
// workgroup owns up to 128 (d = 64) or 64 (d = 128) keys of one key block -- they and their values
// stay in LDS for the whole walk -- and walks the list of ALL
// queries that kept the block (then the block's own queries, causally masked), 32 queries per
// step and wave: the tiles are dense whatever the sequence length, and nothing but the gathered
// query rows and the block's list is read in the loop.
//
// A query's softmax spans several key blocks, i.e. several workgroups.  As in the paper's
// forward each (query, block) pair therefore produces a partial result -- the local softmax
// reference m, the sum l of exp(s - m), and sum p v / l rounded to bf16 -- and a second kernel
// merges a query's partials (Section 4.2: the partial outputs are combined with the
// log-sum-exp weights).  The partials of query t lie together, [t][e][c] for its e-th kept
// block (e = k: own block) and part c of the block's keys, so the merge streams them; e comes with
// the query in the block's list (the list builder files it in the entry's high byte).  No atomics anywhere; results are
// bit-reproducible.
//
// Products of 32 x 32 x 16: S^T of 32 keys and 32 queries leaves a lane with 16 scores of one query, whose
// maximum and sum then cross one lane swap, and the keys are read from LDS once per 32 queries.  The values are
// read through the LDS transpose read straight from their rows, so no transposed copy of V is made, and three
// waves share a SIMD at d = 64 (two at d = 128).  Against products of 16 x 16 x 32 and values in registers from a
// transposed copy: N = 524288, d = 64, B = 128, k = 8, 32 slices: 12.8 + 0.67 (the copy)
// -> 10.2 ms; N = 131072, d = 128, B = 64, k = 32, 16 slices: 7.17 + 0.18 -> 6.59 ms; N = 8192, d = 64, B = 128, k = 8,
// 16 slices: 98 + 7 -> 87 us.  Bounds: the long shapes the scattered 128- and 256-byte rows (queries in, partials
// out: 40 GB in 10.2 ms, 35 GB in 6.6 ms; without the arithmetic 9.4 ms of the first, without the stores 7.0); the
// short ones VALU issue (about 375 instructions per 32 queries x 128 keys) beside the matrix pipe, and how well
// the longest lists fit the end of the launch.
#include <type_traits>

#include "mfma.h"

namespace moba {

template <int D, int NG>                                   // NG: 32-key groups of a workgroup
struct KmCfg {
    static constexpr int NW = 4;
    static constexpr int NT = NW * kWave;
    static constexpr int SB = D * 2 + 16;              // bytes per parked row: 32 rows x 2 pieces meet every bank once
    static constexpr int CT = D / 32;                  // 32-channel tiles of a row
    static constexpr int KS = D / 16;                  // contraction steps of q.k
    static constexpr int CPR = D / 8;                  // 16-byte pieces per row = lanes per gathered row
    static constexpr int RPI = kWave / CPR;            // rows per gather instruction
    static constexpr int NI = 32 / RPI;                // gather instructions per step
    static constexpr size_t PARK = (size_t)NW * 32 * SB;                 // the waves' parked rows
    static constexpr size_t PART = (size_t)NG * 64 * D;                  // bytes of the part's keys (or values)
    static constexpr size_t LDS = PARK + 2 * PART;
};

template <int D, int NG>
__global__ __launch_bounds__((KmCfg<D, NG>::NT)) __attribute__((amdgpu_waves_per_eu(D == 64 ? 3 : 2)))
void fwd_km_kernel(
    const bf16_t* __restrict__ Q, const bf16_t* __restrict__ K, const bf16_t* __restrict__ V,
    const int32_t* __restrict__ off, const int32_t* __restrict__ ql,
    bf16_t* __restrict__ PO, float* __restrict__ Pml, int N, int B, int n, int k, int nsub,
    float scale, int64_t R, int bh, int G, int inter)
{
    using C = KmCfg<D, NG>;
    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid / kWave), lane = tid % kWave;
    const int m32 = lane & 31, h = lane >> 5;
    unsigned char* stQ = smem + (size_t)wave * 32 * C::SB;
    unsigned char* sK = smem + C::PARK;
    unsigned char* sV = sK + C::PART;

    int s, u;                                               // slice, (key block, part)
    if (!schedule(blockIdx.x, bh, n * nsub, s, u, inter)) return;
    const int j = u / nsub, c = u - j * nsub;
    const int own_first = c * (32 * NG);                    // first key of the part inside the block
    const int64_t sbase = (int64_t)s * N;
    const int64_t kvbase = (int64_t)(s / G) * N;            // G query heads share a key/value head
    const float c2 = scale * kLog2e;
    const int32_t* os = off + (int64_t)s * (n + 1);
    const int32_t* qs = ql + (int64_t)s * R;
    const int lo = os[j], nlist = os[j + 1] - lo;
    const int own0 = j * B + own_first;                     // own queries that see keys of this part
    const int total = nlist + (B - own_first);
    const char* Qg = reinterpret_cast<const char*>(Q + sbase * D);

    // Every load of the walk is unconditional and from an address that is always valid (a load
    // inside a branch is waited for at the end of the branch).
    // Position a of the walk -> list entry (query, e); own rows and rows past the end: e = k.
    const int32_t* lsrc = nlist > 0 ? qs + lo : os;
    const int llast = max(nlist - 1, 0);
    const int own_e = k << 24;
    auto query_at = [&](int a) {
        const int listed = lsrc[min(a, llast)];
        const int t = a < nlist ? listed : (own0 + (a - nlist)) | own_e;
        return a >= total ? own0 | own_e : t;
    };
    const int grow = lane / C::CPR;                         // row of this lane inside a gather instruction
    const uint32_t gcol = (uint32_t)(lane % C::CPR) * 16u;  // its 16-byte piece of the row
    // t: rows this lane gathers a piece of; tl: row m32.  `inside` (a compile-time flag): all these
    // positions lie in the block's list -- the bulk of the walk, which then needs no selects
    auto ids = [&](int a0, int (&t)[C::NI], int& tl, auto inside) {
        if constexpr (decltype(inside)::value) {
#pragma unroll
            for (int i = 0; i < C::NI; ++i) t[i] = lsrc[a0 + C::RPI * i + grow];
            tl = lsrc[a0 + m32];
        } else {
#pragma unroll
            for (int i = 0; i < C::NI; ++i) t[i] = query_at(a0 + C::RPI * i + grow);
            tl = query_at(a0 + m32);
        }
    };
    auto fetch = [&](const int (&t)[C::NI], u32x4_t (&qr)[C::NI]) {
#pragma unroll
        for (int i = 0; i < C::NI; ++i)
            qr[i] = *reinterpret_cast<const u32x4_t*>(Qg + (uint32_t)list_query(t[i]) * (uint32_t)(2 * D) + gcol);
    };
    // The rows of the next step are in flight while a step is worked on, the list entries of the one
    // after it too: tc, tlc name the rows in qr, tn, tln those of the step after.
    constexpr int stride = 32 * C::NW;
    int tc[C::NI], tn[C::NI], tlc, tln;
    u32x4_t qr[C::NI];
    ids(32 * wave, tc, tlc, std::false_type());
    ids(32 * wave + stride, tn, tln, std::false_type());
    fetch(tc, qr);

    // The part's keys go to LDS in MFMA operand order -- the 16 bytes lane (m, h) feeds as row m,
    // channels 16 ks + 8 h .. + 8 of 32-key group gi sit at (gi * KS + ks) * 1024 + 16 * lane --, its
    // values as rows, 64-byte quarters (d = 64: halves) of row r permuted by r & 3 (r >> 1 & 1): the
    // transpose reads below take four rows' 64 bytes at a time and so meet every bank once.  All values are requested before the
    // first one is waited for, then all keys: one 16-byte piece of each after the other left a workgroup waiting for them in turn, and
    // both together made a launch whose values come from HBM (the centroids have read the keys before) slower.  Whole step of 18 slices
    // of 10080 (B = 96, k = 10), inputs cold: in turn 487, together 480, keys first 479, values first 473 us; forward and routing of
    // 16 slices of 8192: 150.2, 153.9, 152.7, 149.7 us.  One piece of each (d = 64, B = 32) comes at once: 12 slices of 38848, k = 8,
    // kernel 255 us, values first 271.
    {
        const char* Kg = reinterpret_cast<const char*>(K + (kvbase + own0) * D);
        const char* Vg = reinterpret_cast<const char*>(V + (kvbase + own0) * D);
        constexpr int IT = NG * 32 * C::CPR / C::NT;
        u32x4_t vr[IT], kr[IT];
#pragma unroll
        for (int i = 0; i < IT; ++i) vr[i] = *reinterpret_cast<const u32x4_t*>(Vg + (size_t)(i * C::NT + tid) * 16);
        if constexpr (IT == 1) kr[0] = *reinterpret_cast<const u32x4_t*>(Kg + (size_t)tid * 16);
#pragma unroll
        for (int i = 0; i < IT; ++i) {
            const int row = (i * C::NT + tid) / C::CPR, col = (i * C::NT + tid) % C::CPR;   // key of the part, 16-byte piece
            const int sx = D == 64 ? (row >> 1) & 1 : row & 3;
            *reinterpret_cast<u32x4_t*>(sV + row * 2 * D + (col ^ (sx << 2)) * 16) = vr[i];
        }
        if constexpr (IT > 1) {
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < IT; ++i) kr[i] = *reinterpret_cast<const u32x4_t*>(Kg + (size_t)(i * C::NT + tid) * 16);
        }
#pragma unroll
        for (int i = 0; i < IT; ++i) {
            const int row = (i * C::NT + tid) / C::CPR, col = (i * C::NT + tid) % C::CPR;
            *reinterpret_cast<u32x4_t*>(sK + ((row >> 5) * C::KS + (col >> 1)) * 1024 + ((col & 1) * 32 + (row & 31)) * 16) = kr[i];
        }
    }
    __syncthreads();

    // Transpose reads: lanes 4 e + a of a 16-lane group point at key row 4 h + e, 8-byte piece a of the
    // group's 16 channels (lanes 16 .. 31 of a half: the upper sixteen of a 32-channel tile)
    const unsigned char* vt[C::CT];
    {
        const int e = (lane >> 2) & 3, sx = D == 64 ? e >> 1 : e;
#pragma unroll
        for (int ct = 0; ct < C::CT; ++ct)
            vt[ct] = sV + (4 * h + e) * 2 * D + (ct ^ sx) * 64 + ((lane >> 4) & 1) * 32 + (lane & 3) * 8;
    }
    const unsigned char* ka0 = sK + lane * 16;
    const uint32_t slots = (uint32_t)(k + 1) * nsub;        // partials per query
    // (32-bit indices of partials inside a slice: more would not fit the device's memory)
    bf16_t* POs = PO + sbase * slots * D;
    float* Pmls = Pml + sbase * slots * 2;
    // clamped: lists that do not match the rows of kept blocks give a wrong result, never an address
    // outside the partials
    auto partial = [&](int entry) {
        return __umul24(min(list_query(entry), N - 1), slots) + __umul24(min(list_slot(entry), k), nsub) + (uint32_t)c;
    };
    unsigned char* const rowm = stQ + m32 * C::SB;

    auto step = [&](int a0, auto inside) {
        constexpr bool in = decltype(inside)::value;
        int to[C::NI];
#pragma unroll
        for (int i = 0; i < C::NI; ++i) {
            *reinterpret_cast<u32x4_t*>(stQ + (C::RPI * i + grow) * C::SB + gcol) = qr[i];
            to[i] = tc[i];
            tc[i] = tn[i];
        }
        const int tlo = tlc;
        tlc = tln;
        fetch(tc, qr);
        ids(a0 + 2 * stride, tn, tln, inside);
        __builtin_amdgcn_wave_barrier();
        Frag qb[C::KS];
#pragma unroll
        for (int ks = 0; ks < C::KS; ++ks) qb[ks].q = *reinterpret_cast<const uint4*>(rowm + 32 * ks + 16 * h);
        // raw scores of row m32 against the part's keys: x[gi][i] is key 32 gi + 8 (i >> 2) + 4 h + (i & 3).
        // (The scheduling barriers here and below keep the LDS reads of the next products ahead of the
        // current ones; left alone, the compiler reads an operand right before it is used and waits.)
        f32x16_t x[NG];
        Frag ka[2][C::KS];
        auto keys = [&](int gi) {
#pragma unroll
            for (int ks = 0; ks < C::KS; ++ks)
                ka[gi & 1][ks].q = *reinterpret_cast<const uint4*>(ka0 + (gi * C::KS + ks) * 1024);
        };
        keys(0);
#pragma unroll
        for (int gi = 0; gi < NG; ++gi) {
            if (gi + 1 < NG) keys(gi + 1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < 16; ++i) x[gi][i] = 0.f;
#pragma unroll
            for (int ks = 0; ks < C::KS; ++ks) x[gi] = mfma32(ka[gi & 1][ks], qb[ks], x[gi]);
            __builtin_amdgcn_sched_barrier(0);
        }
        if (!in && a0 + 32 > nlist) {                              // own row r sees keys 0 .. r of the part
            const int r = a0 + m32 - nlist, last = (r >= 0 ? r : 32 * NG) - 4 * h;
#pragma unroll
            for (int gi = 0; gi < NG; ++gi)
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    if (32 * gi + 8 * (i >> 2) + (i & 3) > last) x[gi][i] = -INFINITY;
        }
        float mref = x[0][0];
#pragma unroll
        for (int gi = 0; gi < NG; ++gi)
#pragma unroll
            for (int i = 0; i < 16; ++i) mref = max_nan(mref, x[gi][i]);
        mref = max_halves(mref) * c2;               // c2 > 0: the maximum commutes
        // p of 16 keys at a time, ahead of their products with the values
        float l = 0.f;
        Frag pb[2], va[2][C::CT];
        auto probabilities = [&](int it) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int i = 8 * (it & 1) + 2 * e;
                const float p0 = fast_exp2(fmaf(x[it >> 1][i], c2, -mref)), p1 = fast_exp2(fmaf(x[it >> 1][i + 1], c2, -mref));
                l += p0;
                l += p1;
                pb[it & 1].u[e] = pack2(p0, p1);
            }
        };
        auto values = [&](int it) {
#pragma unroll
            for (int ct = 0; ct < C::CT; ++ct) {
                const unsigned char* v = vt[ct] + 16 * it * 2 * D;
                const uint2 v0 = lds_read_tr16(v), v1 = lds_read_tr16(v + 16 * D);
                va[it & 1][ct].u[0] = v0.x; va[it & 1][ct].u[1] = v0.y;
                va[it & 1][ct].u[2] = v1.x; va[it & 1][ct].u[3] = v1.y;
            }
        };
        f32x16_t o[C::CT];
        values(0);
        __builtin_amdgcn_sched_barrier(0);
        probabilities(0);
#pragma unroll
        for (int ct = 0; ct < C::CT; ++ct)
#pragma unroll
            for (int i = 0; i < 16; ++i) o[ct][i] = 0.f;
#pragma unroll
        for (int it = 0; it < 2 * NG; ++it) {
            if (it + 1 < 2 * NG) values(it + 1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int ct = 0; ct < C::CT; ++ct) o[ct] = mfma32(va[it & 1][ct], pb[it & 1], o[ct]);
            if (it + 1 < 2 * NG) probabilities(it + 1);
            __builtin_amdgcn_sched_barrier(0);
        }
        l = sum_halves(l);
        // The partial: this lane holds channels 32 ct + 8 q4 + 4 h .. + 4 of row m32.  It goes back over
        // the row's parked bytes (the Q operands are in registers by now) and is then written out by
        // whole rows -- CPR neighbouring lanes store one row's 2 D consecutive bytes, so every line of
        // the partials is written by one instruction.
        // (normalised before it is rounded: where one partial outweighs the rest, the merge then gives its
        // rounded values back, and the result is rounded once, not twice; a correctly rounded reciprocal instead of
        // v_rcp_f32: 16 slices of N = 8192, B = 128 93.2 -> 93.7 us, of 131072, d = 128, B = 64, k = 32 9838 both)
        const float inv = 1.f / l;
#pragma unroll
        for (int ct = 0; ct < C::CT; ++ct)
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4)
                *reinterpret_cast<uint2*>(rowm + 64 * ct + 16 * q4 + 8 * h) =
                    make_uint2(pack_bf16x2(o[ct][4 * q4] * inv, o[ct][4 * q4 + 1] * inv),
                               pack_bf16x2(o[ct][4 * q4 + 2] * inv, o[ct][4 * q4 + 3] * inv));
        __builtin_amdgcn_wave_barrier();
        u32x4_t out[C::NI];
#pragma unroll
        for (int i = 0; i < C::NI; ++i)
            out[i] = *reinterpret_cast<const u32x4_t*>(stQ + (C::RPI * i + grow) * C::SB + gcol);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < C::NI; ++i) {
            if (in || a0 + C::RPI * i + grow < total) {
                u32x4_t* dst = reinterpret_cast<u32x4_t*>(reinterpret_cast<char*>(POs + (uint64_t)partial(to[i]) * D) + gcol);
                // d = 128: streaming stores -- the partials are read again only by the merge
                // kernel, and not keeping their two lines per row in L2 measured -17 % there
                // (d = 64: no difference)
                if constexpr (D == 128) __builtin_nontemporal_store(out[i], dst);
                else *dst = out[i];
            }
        }
        // (m, l) of the step's 32 rows in one store instruction, a lane per row
        if (h == 0 && (in || a0 + m32 < total)) {
            typedef float f32x2_t __attribute__((ext_vector_type(2)));
            f32x2_t* pm = reinterpret_cast<f32x2_t*>(Pmls + (uint64_t)partial(tlo) * 2);
            const f32x2_t ml = {mref, l};
            if constexpr (D == 128) __builtin_nontemporal_store(ml, pm);
            else *pm = ml;
        }
        __builtin_amdgcn_wave_barrier();
    };
    // the bulk of the walk: this step, the rows fetched in it and the entries looked up in it all lie
    // inside the block's list; then the general steps (own rows, causal mask, end of the walk)
    int a0 = 32 * wave;
    for (; a0 + 2 * stride + 32 <= nlist; a0 += stride) step(a0, std::true_type());
    for (; a0 < total; a0 += stride) step(a0, std::false_type());
}

// O_t = sum w O_p / L, w = l_p 2^(m_p - M), L = sum w, over the query's partials: all parts of its kept
// blocks, and the parts of its own block up to its own key; lse_t = (M + log2 L) ln 2.
// One pass: the reference M is that of the chunks so far, and the sums are scaled when it moves.
template <int D, int CH>
__global__ __launch_bounds__(256) void fwd_km_merge_kernel(
    const int32_t* __restrict__ idx, const bf16_t* __restrict__ PO, const float* __restrict__ Pml,
    bf16_t* __restrict__ O, float* __restrict__ lse, int N, int B, int k, int nsub)
{
    using R = MergeRow<D>;
    constexpr int PER = (CH + R::LANES - 1) / R::LANES;          // partials of a chunk a lane looks up
    const R r(idx, N, B, k, nsub, km_part_keys(B, D));
    const float2* mlrow = reinterpret_cast<const float2*>(Pml) + r.row * r.slots;
    const char* orow = reinterpret_cast<const char*>(PO + r.row * r.slots * D + r.piece * 8);
    float M = -INFINITY, L = 0.f, acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    for (int i0 = 0; i0 < r.slots; i0 += CH) {
        u32x4_t raw[CH];
        float2 ml[PER];
        bool ok[PER];
#pragma unroll
        for (int p = 0; p < PER; ++p) {
            const int at = p * R::LANES + r.piece, si = i0 + at;
            ml[p] = mlrow[min(si, r.slots - 1)];
            ok[p] = r.counts(si) && at < CH;
        }
#pragma unroll
        for (int i = 0; i < CH; ++i)
            raw[i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(orow + (int64_t)min(i0 + i, r.slots - 1) * (2 * D)));
        float top = M;
#pragma unroll
        for (int p = 0; p < PER; ++p) top = fmaxf(top, ok[p] ? ml[p].x : -INFINITY);
#pragma unroll
        for (int o = 1; o < R::LANES; o <<= 1) top = fmaxf(top, __shfl_xor(top, o, kWave));
        const float ref = top == -INFINITY ? 0.f : top;          // (no partial yet: all weights are zero)
        const float turn = fast_exp2(M - ref);
        M = top;
        L *= turn;
#pragma unroll
        for (int ch = 0; ch < 8; ++ch) acc[ch] *= turn;
        float w[PER];
#pragma unroll
        for (int p = 0; p < PER; ++p) {
            w[p] = ok[p] ? ml[p].y * fast_exp2(ml[p].x - ref) : -1.f;      // -1: not there
            L += ok[p] ? w[p] : 0.f;                             // (this lane's partials)
        }
        unrolled(std::make_integer_sequence<int, CH>{}, [&](auto i_) {
            constexpr int i = decltype(i_)::value;
            const float wi = from_lane_of_group<R::LANES, i % R::LANES>(w[i / R::LANES]);
            // (an unused slot holds whatever the workspace held: select, do not multiply by 0)
            const bool unused = wi < 0.f;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint32_t x = unused ? 0u : raw[i][q];
                acc[2 * q] = fmaf(wi, __uint_as_float(x << 16), acc[2 * q]);
                acc[2 * q + 1] = fmaf(wi, __uint_as_float(x & 0xffff0000u), acc[2 * q + 1]);
            }
        });
    }
#pragma unroll
    for (int o = 1; o < R::LANES; o <<= 1) L += __shfl_xor(L, o, kWave);
    const float inv = 1.f / L;
#pragma unroll
    for (int ch = 0; ch < 8; ++ch) acc[ch] *= inv;
    Vec8<bf16_t>::store(O + r.row * D + r.piece * 8, acc);
    if (r.piece == 0) lse[r.row] = (M + fast_log2(L)) * kLn2;
}

// ---- workspace: [partial O: bh*N*(k+1)*parts*D bf16][partial (m, l): bh*N*(k+1)*parts*2 fp32],
// each 256-byte aligned.  (And the size of V, which nothing uses any more: what moba_workspace_bytes reports for a
// shape, and that sharing key/value heads lowers it, stays as it was.)

size_t forward_km_ws_bytes(const Dims& s)
{
    const size_t tensor = a256(sizeof(bf16_t) * (size_t)s.bhk * s.N * s.D);
    return tensor + a256(sizeof(bf16_t) * km_partials(s) * s.D) + a256(sizeof(float) * km_partials(s) * 2);
}

template <int D, int NG>
static hipError_t km_launch2(const Dims& s, const void* Q, const void* K, const void* V,
                             const int32_t* idx, const int32_t* off, const int32_t* ql, bf16_t* PO,
                             float* Pml, void* O, float* lse, hipStream_t st)
{
    using C = KmCfg<D, NG>;
    const int nsub = s.B / km_part_keys(s.B, s.D);
    hipError_t e = ensure_dynamic_lds((const void*)fwd_km_kernel<D, NG>, C::LDS);
    if (e != hipSuccess) return e;
    {
        ProfileScope timing(MOBA_PROFILE_FORWARD, st);
        const int bhs = slice_major(s, 1) * s.bh;           // (gathers Q rows)
        hipLaunchKernelGGL((fwd_km_kernel<D, NG>), dim3((unsigned)schedule_grid(bhs, s.n * nsub)),
                           dim3(C::NT), C::LDS, st, (const bf16_t*)Q, (const bf16_t*)K, (const bf16_t*)V,
                           off, ql, PO, Pml, s.N, s.B, s.n, s.k, nsub, s.scale, s.R, bhs, s.G, interleave(s, 1));
    }
    const dim3 grid((unsigned)((int64_t)s.bh * s.N / MergeRow<D>::ROWS));
#define MOBA_MERGE(CH)                                                                                              \
    hipLaunchKernelGGL((fwd_km_merge_kernel<D, CH>), grid, dim3(256), 0, st, idx, PO, Pml, (bf16_t*)O, lse, s.N, s.B, \
                       s.k, nsub);                                                                                  \
    break
    switch (merge_chunk((s.k + 1) * nsub)) {
        case 4: MOBA_MERGE(4);
        case 6: MOBA_MERGE(6);
        case 9: MOBA_MERGE(9);
        case 11: MOBA_MERGE(11);
        default: MOBA_MERGE(13);
    }
#undef MOBA_MERGE
    return hipGetLastError();
}

template <int D, typename... A>
static hipError_t km_launch(const Dims& s, A... a)
{
    switch (km_part_keys(s.B, D) / 32) {
        case 1: return km_launch2<D, 1>(s, a...);
        case 2: return km_launch2<D, 2>(s, a...);
        case 3: if constexpr (D == 64) return km_launch2<D, 3>(s, a...); else break;
        case 4: if constexpr (D == 64) return km_launch2<D, 4>(s, a...); else break;
    }
    return hipErrorInvalidValue;
}

hipError_t launch_forward_km(const Dims& s, const void* Q, const void* K, const void* V, void* ws,
                             const int32_t* idx, const int32_t* off, const int32_t* ql, void* O,
                             float* lse, hipStream_t st)
{
    if (s.bh == 0 || s.N == 0) return hipSuccess;
    if (!key_major_shape(s)) return hipErrorInvalidValue;
    char* p = static_cast<char*>(ws);
    bf16_t* PO = reinterpret_cast<bf16_t*>(p);
    p += a256(sizeof(bf16_t) * km_partials(s) * s.D);
    float* Pml = reinterpret_cast<float*>(p);
    return s.D == 64 ? km_launch<64>(s, Q, K, V, idx, off, ql, PO, Pml, O, lse, st)
                     : km_launch<128>(s, Q, K, V, idx, off, ql, PO, Pml, O, lse, st);
}

}  // namespace moba
