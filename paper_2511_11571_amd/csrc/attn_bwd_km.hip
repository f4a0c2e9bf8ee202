// The MoBA backward, key-block major, for sparse routing (paper Section 4.2 backward and Appendix C.3:
// key blocks outermost, the queries routed to a block gathered into dense tiles, S recomputed,
// dV += P^T dO, dS = P o (dP - D), dK += dS^T Q, dQ += scale dS K).  A workgroup owns up to 128 keys of one
// key block, 32 per wave, and walks the block's query list, then the block's own queries (causally masked).
//
// The paper's kernel adds each block's contribution to dQ with atomic additions into a high-precision
// buffer.  Here the contribution of (query t, kept block e, part c) is written once, as bf16, to [t][e][c],
// and a second kernel adds a query's contributions up in fp32 in a fixed order: no atomics,
// bit-reproducible, and the partial sums stream.
//
// Per step of P positions of the walk (NSLOT slots of 32):
//   gather     every wave brings its share of the rows of Q and dO, whole rows per load instruction, ids two
//              steps and rows one step ahead, and parks them in LDS;
//   S, dP      queries x the wave's 32 keys; a lane holds one key and four queries of every 16-query tile,
//              which packed to bf16 is the B operand of
//   dV^T, dK^T += dO^T P, Q^T dS    (the parked rows through the LDS transpose read), in registers for the
//              whole walk, and goes to LDS as dS[key][query];
//   dQ^T = K^T dS^T    over all keys of the workgroup, the step's queries and channels dealt to the waves;
//              both operands through the transpose read.
//
// One walk for all three gradients: dQ on its own repeats the gather of Q and dO and the products S and dP
// (5 products instead of 7).  No pipe is full: at N = 65536, d = 64, B = 128, k = 8, 32 slices the LDS pipe is
// busy 64 % of the clocks, VALU issue 41 %, the matrix pipe 38 % (N = 16384, d = 128, B = 64, k = 16: 43, 26 and 25 %); the latencies of two
// waves per SIMD (d = 64), one (d = 128) are what is left.  Neither whole-line nor streaming stores of the partials nor rows
// gathered from one place make much of a difference there (17.9 -> 17.6 and 16.4 ms).
// Against separate walks for dQ and for dK and dV: N = 524288: 28.0 -> 18.6 ms, with the rows laid out as
// parked() says 17.9; N = 10080, B = 96, k = 10, 18 slices: 210 us; N = 16384, d = 128, B = 64, k = 16, 16 slices: 778 us,
// with that and operands read ahead 705.  Keys requested together, and kept for dQ where there are registers: whole backward
// 22.96 -> 22.20 ms, 235 -> 230 us, 927 -> 894 us.
//
// Tried and left: a third wave per SIMD at d = 64 (LDS rows without padding fit three workgroups, 168 registers do not hold
// the gathered rows: spills, 40 ms instead of 18); a slot's exponentials between the next one's products, with scheduling
// barriers (22.3 -> 23.8 ms); list entries requested before the keys (slower at d = 128).
#include <type_traits>

#include "mfma.h"

namespace moba {

// keys per workgroup: blocks up to 128 whole, larger ones in parts
__host__ __device__ inline int bwd_part_keys(int B, int D)
{
    return B <= km_part_keys(B, D) ? B : B % 128 == 0 ? 128 : 64;
}

// rows in LDS, by 16-byte pieces: row-major operand reads (16 rows at one piece; the 16 lanes served together are
// 0-3, 12-15 and 20-27, i.e. rows 0-3 and 12-15 at one piece and rows 4-11 at the next) and transpose reads (8
// rows at two neighbouring pieces) both meet every bank once: 4 and 3 clocks per instruction.  (Rows of 144
// bytes: 8 and 4; a piece XORed with the row rotated by one: 8 and 3.)  d = 64: padded rows; d = 128: the piece XORed
// with bits of the row.
template <int D>
__device__ __forceinline__ uint32_t parked(uint32_t row, uint32_t piece)
{
    if constexpr (D == 64) return row * 160u + piece * 16u;
    const uint32_t r = row, x = (r >> 3 & 1u) | (r & 3u) << 1 | ((r >> 2 ^ r >> 3) & 1u) << 3;
    return row * 256u + ((piece ^ x) * 16u);
}

template <int D, int NG>                               // NG: 32-key groups of a workgroup
struct BwdKmCfg {
    static constexpr int NW = NG, NT = NW * kWave;
    static constexpr int NSLOT = NG == 4 ? 2 : NG;      // (four waves park 16 rows each: registers)
    static constexpr int HV = NW / NSLOT;               // waves that share the dQ of a slot, by channels
    static constexpr int P = 32 * NSLOT;                // positions of the walk per step
    static constexpr int MT = D / 16, KS = D / 32;
    static constexpr int CPR = D / 8;                   // 16-byte pieces per row = lanes per gathered row
    static constexpr int RPI = kWave / CPR;             // rows per gather instruction
    static constexpr int RW = P / NW, NI = RW / RPI;    // rows a wave gathers, instructions per tensor
    static constexpr int CH = D / HV, MQ = CH / 16;     // channels and tiles of a wave's share of dQ
    static constexpr int SB = D == 64 ? 160 : 256;      // bytes per parked row
    static constexpr int SLOT = 64 * SB + 3 * 32 * 4;   // Q rows, dO rows, lse, -D, list entry
    static constexpr int XS = 2 * P + 8;                // bytes per key of dS (written by 16 rows at a time: every bank once)
    static constexpr int EX = 32 * NG * XS, KR = 32 * NG * SB;
    static constexpr int RST = D + 4;                   // floats per key row when dK and dV are turned over
    static constexpr size_t WALK = (size_t)NSLOT * SLOT + EX + KR, TURN = (size_t)NW * 32 * RST * 4;
    static constexpr size_t LDS = WALK > TURN ? WALK : TURN;
};

// KV = false: dQ only (a caller that takes the gradients one call at a time), without dV += P^T dO, dK += dS^T Q
template <int D, int NG, bool KV>
__global__ __launch_bounds__((BwdKmCfg<D, NG>::NT)) __attribute__((amdgpu_waves_per_eu(D == 64 ? 2 : 1)))
void bwd_km_kernel(
    const bf16_t* __restrict__ Q, const bf16_t* __restrict__ K, const bf16_t* __restrict__ V,
    const bf16_t* __restrict__ dO, const float2* __restrict__ ld, const int32_t* __restrict__ off,
    const int32_t* __restrict__ ql, bf16_t* __restrict__ dK, bf16_t* __restrict__ dV, bf16_t* __restrict__ PdQ,
    float* __restrict__ part, int N, int B, int n, int k, int nsub, float scale, int64_t R, int order, int bh, int G,
    int inter)
{
    using C = BwdKmCfg<D, NG>;
    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid / kWave), lane = tid % kWave;
    const int m16 = lane & 15, g = lane >> 4;
    unsigned char* ex = smem + C::NSLOT * C::SLOT;          // dS[key][query of the step]
    unsigned char* sK = ex + C::EX;                         // the part's K rows, for dQ

    int s, u;                                               // query slice, (key block, part)
    if (!schedule(blockIdx.x, order * bh, n * nsub, s, u, inter)) return;
    const int j = u / nsub, c = u - j * nsub;
    const int own_first = c * (32 * NG);                    // first key of the part inside the block
    const int own0 = j * B + own_first;                     // ... of the slice; own queries that see keys of this part
    const int kfirst = 32 * wave;                           // this wave's first key inside the part
    const int64_t sbase = (int64_t)s * N;
    const int64_t kvbase = (int64_t)(s / G) * N;            // G query heads share a key/value head
    const float c2 = scale * kLog2e;
    const int32_t* os = off + (int64_t)s * (n + 1);
    const int32_t* qs = ql + (int64_t)s * R;
    const int lo = os[j], nlist = os[j + 1] - lo;
    const int total = nlist + (B - own_first);
    const char* Qg = reinterpret_cast<const char*>(Q + sbase * D);
    const char* Gg = reinterpret_cast<const char*>(dO + sbase * D);

    // The K rows of the part, their 8-byte pieces (four channels) in the order in which dQ's transpose reads
    // want them: a lane of the result then holds CH / 4 consecutive channels.  All are requested before the first one is
    // waited for: one after the other they took most of the 14000 clocks (of 122000) before a workgroup's walk.
    {
        const char* Kg = reinterpret_cast<const char*>(K + (kvbase + own0) * D);
        constexpr int KI = 32 * NG * C::CPR / C::NT;
        uint4 krow[KI];
#pragma unroll
        for (int i = 0; i < KI; ++i) krow[i] = *reinterpret_cast<const uint4*>(Kg + (size_t)(i * C::NT + tid) * 16);
#pragma unroll
        for (int i = 0; i < KI; ++i) {
            const int row = (i * C::NT + tid) / C::CPR, piece = (i * C::NT + tid) % C::CPR;
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const int ch = 2 * piece + e, half = ch / (C::CH / 4), in = ch % (C::CH / 4);
                const int pos = half * (C::CH / 4) + 4 * (in % C::MQ) + in / C::MQ;
                *reinterpret_cast<uint2*>(sK + parked<D>(row, pos >> 1) + 8 * (pos & 1)) =
                    e ? make_uint2(krow[i].z, krow[i].w) : make_uint2(krow[i].x, krow[i].y);
            }
        }
    }
    // B operands: the wave's keys and values (lane = key m16 of tile nt)
    Frag kb[2][C::KS], vb[2][C::KS];
#pragma unroll
    for (int nt = 0; nt < 2; ++nt)
#pragma unroll
        for (int ks = 0; ks < C::KS; ++ks) {
            const int64_t o = (kvbase + own0 + kfirst + 16 * nt + m16) * D + 8 * g + 32 * ks;
            kb[nt][ks].q = *reinterpret_cast<const uint4*>(K + o);
            vb[nt][ks].q = *reinterpret_cast<const uint4*>(V + o);
        }
    f32x4_t dKT[C::MT][2], dVT[C::MT][2];
#pragma unroll
    for (int mt = 0; mt < C::MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) {
            dKT[mt][nt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
            dVT[mt][nt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        }

    // position a of the walk -> list entry (query, e: the place of this block in the query's row of kept
    // blocks, filed in the entry's high byte by the list builder); own rows and rows past the end: e = k.
    // Every load of the walk is unconditional and from an address that is always valid (a load inside a
    // branch would be waited for at the end of the branch).
    const int32_t* lsrc = nlist > 0 ? qs + lo : os;
    const int llast = max(nlist - 1, 0);
    const int own_e = k << 24;
    auto query_at = [&](int a) {
        const int listed = lsrc[min(a, llast)];
        const int t = a < nlist ? listed : (own0 + (a - nlist)) | own_e;
        return a >= total ? own0 | own_e : t;
    };
    const int grow = lane / C::CPR;                          // row of this lane inside a gather instruction
    const uint32_t gcol = (uint32_t)(lane % C::CPR);         // its 16-byte piece of the row
    const int first = C::RW * wave;                          // this wave's rows inside a step
    // `inside` (a compile-time flag): all positions lie in the block's list -- the bulk of the walk, which
    // then needs no selects.  t: rows this lane gathers a piece of; tl: the row whose lse, D and entry it brings
    auto ids = [&](int a0, int (&t)[C::NI], int& tl, auto inside) {
        const int a = a0 + first;
        if constexpr (decltype(inside)::value) {
#pragma unroll
            for (int i = 0; i < C::NI; ++i) t[i] = lsrc[a + C::RPI * i + grow];
            tl = lsrc[a + (lane & (C::RW - 1))];
        } else {
#pragma unroll
            for (int i = 0; i < C::NI; ++i) t[i] = query_at(a + C::RPI * i + grow);
            tl = query_at(a + (lane & (C::RW - 1)));
        }
    };
    // lv: lse in log2 units (+inf past the end: P = 0); dv: -D, the start value of the dP product
    auto fetch = [&](int a0, const int (&t)[C::NI], int tl, u32x4_t (&qr)[C::NI], u32x4_t (&gr)[C::NI],
                     float& lv, float& dv, auto inside) {
#pragma unroll
        for (int i = 0; i < C::NI; ++i) {
            const uint32_t o = (uint32_t)list_query(t[i]) * (uint32_t)(2 * D) + gcol * 16u;
            qr[i] = *reinterpret_cast<const u32x4_t*>(Qg + o);
            gr[i] = *reinterpret_cast<const u32x4_t*>(Gg + o);
        }
        const bool live = decltype(inside)::value || a0 + first + (lane & (C::RW - 1)) < total;
        const float2 x = ld[sbase + list_query(tl)];          // (lse log2 e, -D) of the row
        lv = live ? x.x : INFINITY;
        dv = live ? x.y : 0.f;
    };
    int tN[C::NI], tlN, tl;
    u32x4_t qr[C::NI], gr[C::NI];    // plain vectors: a struct type would be copied through scratch
    float lv, dv;
    {
        int t0[C::NI];
        ids(0, t0, tl, std::false_type());
        fetch(0, t0, tl, qr, gr, lv, dv, std::false_type());
        ids(C::P, tN, tlN, std::false_type());
    }
    // the wave's parked rows; row-major operand of this lane; its pointers of the transpose reads (lanes
    // 4 e + a of a 16-lane group point at contraction row e (+4: 16 rows on), 8-byte piece a)
    unsigned char* mine = smem + (first / 32) * C::SLOT;
    const int row0 = first % 32;
    const int te = (lane >> 2) & 3, ta = lane & 3;
    const uint32_t trow = (uint32_t)slot_key(g, te);
    static_assert(slot_key(0, 4) == slot_key(0, 0) + 16, "the second half of a transpose read: 16 rows on");
    auto tr = [&](const unsigned char* rows, int piece8) {   // A operand: 32 rows as contraction, pieces piece8 + (0 .. 3)
        const uint32_t p = (uint32_t)piece8 + ta, o = parked<D>(trow, p >> 1) + 8u * (p & 1u);
        const uint2 a = lds_read_tr16(rows + o), b = lds_read_tr16(rows + o + 16 * C::SB);
        Frag f;
        f.u[0] = a.x; f.u[1] = a.y; f.u[2] = b.x; f.u[3] = b.y;
        return f;
    };
    const uint32_t exw = (uint32_t)(kfirst + m16) * C::XS + 8u * g;
    const uint32_t exr = trow * C::XS + 8u * ta;
    const int dslot = wave / C::HV, dhalf = wave % C::HV;     // this wave's share of dQ
    const int64_t slots = (int64_t)(k + 1) * nsub;           // partials per query

    // dQ's operand of K: 32 keys as contraction, channel tile it mod MQ of the wave's share.  The same in every step:
    // with four key groups at d = 64 there are registers for all of them (16 of 93 LDS instructions of a step)
    constexpr bool KEEP = D == 64 && NG == 4;
    Frag kept[KEEP ? NG * C::MQ : 1];
    auto key_operand = [&](int it) { return tr(sK + 32 * (it / C::MQ) * C::SB, dhalf * (C::CH / 4) + 4 * (it % C::MQ)); };
    auto ahead = [&]() { if constexpr (D == 128) __builtin_amdgcn_sched_barrier(0); };
    // 32 parked positions (walk positions p0 .. p0 + 31) against this wave's keys
    auto work = [&](const unsigned char* stQ, int sl, int p0, auto inside) {
        const unsigned char* stG = stQ + 32 * C::SB;
        const float* ls = reinterpret_cast<const float*>(stQ + 64 * C::SB);
        const float* Ds = ls + 32;
        // d = 128, one wave per SIMD: every operand is read well ahead of its product, with scheduling barriers
        // in between -- left alone, the compiler reads an operand right before it is used, and the wave waits for
        // it (N = 16384, B = 64, k = 16, 16 slices: 751 -> 705 us).  At d = 64 the second wave fills those waits.
        f32x4_t sc[2][2], dp[2][2], nd[2], l4[2];
        Frag qa[2][C::KS], ga[2][C::KS];
#pragma unroll
        for (int qt = 0; qt < 2; ++qt) {
#pragma unroll
            for (int ks = 0; ks < C::KS; ++ks) {
                const uint32_t o = parked<D>(m16, 4 * ks + g) + qt * 16 * C::SB;
                qa[qt][ks].q = *reinterpret_cast<const uint4*>(stQ + o);
                ga[qt][ks].q = *reinterpret_cast<const uint4*>(stG + o);
            }
            nd[qt] = *reinterpret_cast<const f32x4_t*>(Ds + 16 * qt + 4 * g);   // -D of the rows
            l4[qt] = *reinterpret_cast<const f32x4_t*>(ls + 16 * qt + 4 * g);
        }
        ahead();
#pragma unroll
        for (int qt = 0; qt < 2; ++qt) {
#pragma unroll
            for (int nt = 0; nt < 2; ++nt) {
                sc[qt][nt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
                dp[qt][nt] = nd[qt];                          // dP - D comes out of the MFMA
            }
#pragma unroll
            for (int ks = 0; ks < C::KS; ++ks)
#pragma unroll
                for (int nt = 0; nt < 2; ++nt) {
                    sc[qt][nt] = mfma16(qa[qt][ks], kb[nt][ks], sc[qt][nt]);
                    dp[qt][nt] = mfma16(ga[qt][ks], vb[nt][ks], dp[qt][nt]);
                }
        }
        constexpr int AHEAD = D == 64 ? 1 : 3;                // transposed operands read ahead
        Frag qT[AHEAD + 1], gT[AHEAD + 1];
        auto transposed = [&](int mt) {
            qT[mt % (AHEAD + 1)] = tr(stQ, 4 * mt);
            gT[mt % (AHEAD + 1)] = tr(stG, 4 * mt);
        };
        if (KV) {
#pragma unroll
            for (int mt = 0; mt < AHEAD; ++mt) transposed(mt);
        }
        ahead();
        // own queries are causal: the wave's key kfirst + 16 nt + m16 must not exceed the query
        const bool causal = !decltype(inside)::value && p0 + 32 > nlist && p0 < nlist + kfirst + 32;
        Frag pb[2], sb[2];
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) {
            float p[8], d[8];
#pragma unroll
            for (int qt = 0; qt < 2; ++qt) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    float pv = fast_exp2(fmaf(sc[qt][nt][i], c2, -l4[qt][i]));
                    if (causal) {
                        const int a = p0 + 16 * qt + 4 * g + i - nlist;     // own row index, if >= 0
                        if (a >= 0 && kfirst + 16 * nt + m16 > a) pv = 0.f;
                    }
                    p[4 * qt + i] = pv;
                    d[4 * qt + i] = pv * dp[qt][nt][i];
                }
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                pb[nt].u[e] = pack2(p[2 * e], p[2 * e + 1]);
                sb[nt].u[e] = pack2(d[2 * e], d[2 * e + 1]);
            }
#pragma unroll
            for (int qt = 0; qt < 2; ++qt)
                *reinterpret_cast<uint2*>(ex + exw + 16 * nt * C::XS + 64 * sl + 32 * qt) =
                    make_uint2(sb[nt].u[2 * qt], sb[nt].u[2 * qt + 1]);
        }
#pragma unroll
        for (int mt = 0; KV && mt < C::MT; ++mt) {
            if (mt + AHEAD < C::MT) transposed(mt + AHEAD);
            ahead();
#pragma unroll
            for (int nt = 0; nt < 2; ++nt) {
                dVT[mt][nt] = mfma16(gT[mt % (AHEAD + 1)], pb[nt], dVT[mt][nt]);
                dKT[mt][nt] = mfma16(qT[mt % (AHEAD + 1)], sb[nt], dKT[mt][nt]);
            }
            ahead();
        }
    };
    auto meet = [&]() {
        if constexpr (C::NW > 1) __syncthreads();
        else __builtin_amdgcn_wave_barrier();
    };
    auto step = [&](int a0, auto inside) {
#pragma unroll
        for (int i = 0; i < C::NI; ++i) {
            const uint32_t o = parked<D>(row0 + C::RPI * i + grow, gcol);
            *reinterpret_cast<u32x4_t*>(mine + o) = qr[i];
            *reinterpret_cast<u32x4_t*>(mine + 32 * C::SB + o) = gr[i];
        }
        if (lane < C::RW) {
            float* ls = reinterpret_cast<float*>(mine + 64 * C::SB) + row0 + lane;
            ls[0] = lv;
            ls[32] = dv;
            ls[64] = __int_as_float(tl);
        }
        tl = tlN;
        fetch(a0 + C::P, tN, tl, qr, gr, lv, dv, inside);
        ids(a0 + 2 * C::P, tN, tlN, inside);
        meet();                                              // the step's rows are parked; dS of the last one is read
#pragma unroll
        for (int sl = 0; sl < C::NSLOT; ++sl) work(smem + sl * C::SLOT, sl, a0 + 32 * sl, inside);
        int note[2];
#pragma unroll
        for (int qt = 0; qt < 2; ++qt)
            note[qt] = *reinterpret_cast<const int*>(smem + dslot * C::SLOT + 64 * C::SB + 256 + 4 * (16 * qt + m16));
        // dQ^T = K^T dS^T: key groups outside, channel tiles inside; K's operands KA ahead (they do not
        // wait for the other waves), dS's all at once
        constexpr int KA = D == 64 ? 1 : 4;
        Frag ka[KA + 1], xb[NG][2];
        auto keys = [&](int it) {
            if constexpr (!KEEP) ka[it % (KA + 1)] = key_operand(it);
        };
#pragma unroll
        for (int it = 0; it < KA; ++it) keys(it);
        meet();                                              // dS is whole; the parked rows are read
#pragma unroll
        for (int kg = 0; kg < NG; ++kg)
#pragma unroll
            for (int qt = 0; qt < 2; ++qt) {
                const unsigned char* x = ex + exr + 32 * kg * C::XS + 64 * dslot + 32 * qt;
                const uint2 a = lds_read_tr16(x), b = lds_read_tr16(x + 16 * C::XS);
                xb[kg][qt].u[0] = a.x; xb[kg][qt].u[1] = a.y; xb[kg][qt].u[2] = b.x; xb[kg][qt].u[3] = b.y;
            }
        f32x4_t o[2][C::MQ];
#pragma unroll
        for (int qt = 0; qt < 2; ++qt)
#pragma unroll
            for (int mt = 0; mt < C::MQ; ++mt) o[qt][mt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int it = 0; it < NG * C::MQ; ++it) {
            if (it + KA < NG * C::MQ) keys(it + KA);
            ahead();
#pragma unroll
            for (int qt = 0; qt < 2; ++qt)
                o[qt][it % C::MQ] = mfma16(KEEP ? kept[it] : ka[it % (KA + 1)], xb[it / C::MQ][qt], o[qt][it % C::MQ]);
            ahead();
        }
        // the partials: this lane holds CH / 4 consecutive channels of two rows
#pragma unroll
        for (int qt = 0; qt < 2; ++qt) {
            if (!decltype(inside)::value && a0 + 32 * dslot + 16 * qt + m16 >= total) continue;
            // clamped: lists that do not match the rows of kept blocks give a wrong result, never an
            // address outside the partials
            const int e = min(list_slot(note[qt]), k);
            const int64_t prow = (sbase + min(list_query(note[qt]), N - 1)) * slots + (int64_t)e * nsub + c;
            uint4* dst = reinterpret_cast<uint4*>(PdQ + prow * D + dhalf * C::CH + g * (C::CH / 4));
#pragma unroll
            for (int h = 0; h < C::MQ / 2; ++h)
                dst[h] = make_uint4(pack_bf16x2(o[qt][2 * h][0] * scale, o[qt][2 * h][1] * scale),
                                    pack_bf16x2(o[qt][2 * h][2] * scale, o[qt][2 * h][3] * scale),
                                    pack_bf16x2(o[qt][2 * h + 1][0] * scale, o[qt][2 * h + 1][1] * scale),
                                    pack_bf16x2(o[qt][2 * h + 1][2] * scale, o[qt][2 * h + 1][3] * scale));
        }
    };
    __syncthreads();                                          // K is in LDS
    if constexpr (KEEP) {
#pragma unroll
        for (int it = 0; it < NG * C::MQ; ++it) kept[it] = key_operand(it);
    }
    // the bulk of the walk: this step, the rows fetched in it and the ids looked up in it all lie inside the
    // block's list; then the general steps (own rows, causal mask, end of the walk)
    int a0 = 0;
    for (; a0 + 3 * C::P <= nlist; a0 += C::P) step(a0, std::true_type());
    for (; a0 < total; a0 += C::P) step(a0, std::false_type());

    // every wave has the whole sums of its own 32 keys: turned over in LDS (channels of a key side by side),
    // one tensor after the other, and written out.  part != nullptr (key/value heads shared by G query
    // heads): as fp32 to part[dK | dV][query slice][N][D], for dkdv_heads_kernel to add up
    if (!KV) return;
    __syncthreads();                                          // the walk's LDS is no longer read
    float* red = reinterpret_cast<float*>(smem) + (size_t)wave * 32 * C::RST;
#pragma unroll
    for (int which = 0; which < 2; ++which) {
#pragma unroll
        for (int mt = 0; mt < C::MT; ++mt)
#pragma unroll
            for (int nt = 0; nt < 2; ++nt)
                *reinterpret_cast<f32x4_t*>(red + (16 * nt + m16) * C::RST + 16 * mt + 4 * g) =
                    which == 0 ? dKT[mt][nt] : dVT[mt][nt];
        __builtin_amdgcn_wave_barrier();
#pragma unroll 2
        for (int i = lane; i < 32 * C::CPR; i += kWave) {
            const int key = i / C::CPR, piece = i % C::CPR;
            const float* src = red + key * C::RST + 8 * piece;
            const float mul = which == 0 ? scale : 1.f;
            float v[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = src[e] * mul;
            const int64_t row = own0 + kfirst + key;
            if (part) Vec8<float>::store(part + (((int64_t)which * bh + s) * N + row) * D + 8 * piece, v);
            else Vec8<bf16_t>::store((which == 0 ? dK : dV) + (kvbase + row) * D + 8 * piece, v);
        }
        __builtin_amdgcn_wave_barrier();
    }
}

// dQ_t = sum of the query's partials, in the order [kept block][part], then the parts of its
// own block up to its own key.
template <int D, int CH>
__global__ __launch_bounds__(256) void dq_km_merge_kernel(
    const int32_t* __restrict__ idx, const bf16_t* __restrict__ PdQ, bf16_t* __restrict__ dQ, int N,
    int B, int k, int nsub)
{
    using R = MergeRow<D>;
    constexpr int PER = (CH + R::LANES - 1) / R::LANES;          // partials of a chunk a lane looks up
    const R r(idx, N, B, k, nsub, bwd_part_keys(B, D));
    const char* orow = reinterpret_cast<const char*>(PdQ + r.row * r.slots * D + r.piece * 8);
    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    for (int i0 = 0; i0 < r.slots; i0 += CH) {
        u32x4_t raw[CH];
        uint32_t there[PER];                                     // bit i: the i-th of these partials counts
#pragma unroll
        for (int p = 0; p < PER; ++p) {
            const uint64_t all = __ballot(r.counts(i0 + p * R::LANES + r.piece));
            there[p] = (uint32_t)(r.lane & 32 ? all >> 32 : all) >> (r.lane & 31 & ~(R::LANES - 1));
        }
#pragma unroll
        for (int i = 0; i < CH; ++i)
            raw[i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(orow + (int64_t)min(i0 + i, r.slots - 1) * (2 * D)));
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            // (an unused slot holds whatever the workspace held)
            const uint32_t mask = (uint32_t)-(int)((there[i / R::LANES] >> (i % R::LANES)) & 1u);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint32_t x = raw[i][q] & mask;
                acc[2 * q] += __uint_as_float(x << 16);
                acc[2 * q + 1] += __uint_as_float(x & 0xffff0000u);
            }
        }
    }
    Vec8<bf16_t>::store(dQ + r.row * D + r.piece * 8, acc);
}

// ---- workspace: [D: bh*N fp32][partial dQ: bh*N*(k+1)*parts*D bf16], each 256-byte aligned

size_t backward_km_ws_bytes(const Dims& s)
{
    const size_t partials = (size_t)s.bh * s.N * (size_t)(s.k + 1) * (size_t)(s.B / bwd_part_keys(s.B, s.D));
    return a256(sizeof(float) * (size_t)s.bh * s.N) + a256(sizeof(bf16_t) * partials * s.D);
}

template <int D, int NG, bool KV>
static hipError_t bwd_launch2(const Dims& s, const void* Q, const void* K, const void* V, const void* dO,
                              const float2* ld, const int32_t* idx, const int32_t* off, const int32_t* ql, void* dQ,
                              void* dK, void* dV, bf16_t* PdQ, float* part, hipStream_t st)
{
    using C = BwdKmCfg<D, NG>;
    const int nsub = s.B / (32 * NG);
    hipError_t e = ensure_dynamic_lds((const void*)bwd_km_kernel<D, NG, KV>, C::LDS);
    if (e != hipSuccess) return e;
    {
        ProfileScope timing(KV ? MOBA_PROFILE_DKDV : MOBA_PROFILE_DQ, st);
        const int order = slice_major(s, 2);                // (gathers Q and dO rows)
        hipLaunchKernelGGL((bwd_km_kernel<D, NG, KV>), dim3((unsigned)schedule_grid(order * s.bh, s.n * nsub)), dim3(C::NT),
                           C::LDS, st, (const bf16_t*)Q, (const bf16_t*)K, (const bf16_t*)V, (const bf16_t*)dO, ld, off,
                           ql, (bf16_t*)dK, (bf16_t*)dV, PdQ, part, s.N, s.B, s.n, s.k, nsub, s.scale, s.R, order, s.bh,
                           s.G, interleave(s, 2));
    }
    if (KV && part) {
        e = launch_dkdv_heads(s, part, dK, dV, st);
        if (e != hipSuccess) return e;
    }
    {
        ProfileScope timing(MOBA_PROFILE_DQ, st);
        const dim3 grid((unsigned)((int64_t)s.bh * s.N / MergeRow<D>::ROWS));
#define MOBA_MERGE(CH)                                                                                              \
    hipLaunchKernelGGL((dq_km_merge_kernel<D, CH>), grid, dim3(256), 0, st, idx, PdQ, (bf16_t*)dQ, s.N, s.B, s.k,   \
                       nsub);                                                                                       \
    break
        switch (merge_chunk((s.k + 1) * nsub)) {
            case 4: MOBA_MERGE(4);
            case 6: MOBA_MERGE(6);
            case 9: MOBA_MERGE(9);
            case 11: MOBA_MERGE(11);
            default: MOBA_MERGE(13);
        }
#undef MOBA_MERGE
    }
    return hipGetLastError();
}

// dQ, dK and dV; null dK and dV are not wanted
hipError_t launch_backward_km(const Dims& s, const void* Q, const void* K, const void* V, const void* dO,
                              const float2* ld, const int32_t* idx, const int32_t* off, const int32_t* ql, void* dQ,
                              void* dK, void* dV, float* part, void* ws, hipStream_t st)
{
    if (s.bh == 0 || s.N == 0) return hipSuccess;
    if (!key_major_shape(s)) return hipErrorInvalidValue;
    if (s.G == 1) part = nullptr;
    bf16_t* PdQ = reinterpret_cast<bf16_t*>(static_cast<char*>(ws) + a256(sizeof(float) * (size_t)s.bh * s.N));
#define MOBA_BWD(D, NG)                                                                                            \
    return dK ? bwd_launch2<D, NG, true>(s, Q, K, V, dO, ld, idx, off, ql, dQ, dK, dV, PdQ, part, st)              \
              : bwd_launch2<D, NG, false>(s, Q, K, V, dO, ld, idx, off, ql, dQ, dK, dV, PdQ, part, st)
    switch (s.D + bwd_part_keys(s.B, s.D) / 32) {
        case 64 + 1: MOBA_BWD(64, 1);
        case 64 + 2: MOBA_BWD(64, 2);
        case 64 + 3: MOBA_BWD(64, 3);
        case 64 + 4: MOBA_BWD(64, 4);
        case 128 + 1: MOBA_BWD(128, 1);
        case 128 + 2: MOBA_BWD(128, 2);
        case 128 + 4: MOBA_BWD(128, 4);
    }
#undef MOBA_BWD
    return hipErrorInvalidValue;
}

}  // namespace moba
