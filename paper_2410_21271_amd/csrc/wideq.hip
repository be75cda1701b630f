// The compensated quantised layer for 5 and more tokens, in ONE launch:
//
//      y = x.What^T + (x.A^T).B^T          (Sec. 3 forward equation, Alg. 1 step 7)
//
// A workgroup is eight wavefronts: NWR groups of RW row blocks x NWK ranges of the contraction, for up to TB token
// blocks of 16.  Per step every range advances by one 128-column chunk of x.
//  - x is read row by row (256 contiguous bytes per token: 125 B/ns and compute unit from L2, against 37 when every
//    lane fetches its own 16-byte MFMA fragment from global memory) into registers, PX steps ahead, and goes through
//    LDS, where the wavefronts of a range find their fragments.  With NWR = 1 a chunk belongs to one wavefront: one
//    slot and no barrier (a wavefront's LDS operations are carried out in order); otherwise two slots and one barrier
//    per step.
//  - Stored tiles come straight into the registers of the wavefront that owns the row block, D steps ahead; the rows'
//    group scales and zero-point words wait in LDS, put there before the first step.  Every stored tile is decoded once
//    per workgroup and serves all TB token blocks.  All requests are unconditional plain loads (past the end: the last
//    tile again, never used), so that the compiler's wait counts stay exact.
//  - Arithmetic: integer codes minus zero-point exact in fp16, fp32 accumulation per 128 columns, scaled in fp32; t in
//    fp32, split into a high and a low fp16 part for B's product.
//  - Low-rank path: the launch's first workgroups are producers, one (16 rows of A) x (one of kcn ranges of the
//    contraction) for TB token blocks each; they publish t as (value, epoch + 1) pairs and never wait.  After its
//    backbone every consumer adds the kcn partials of its tokens' t in a fixed order, checks the tags, re-reads past the
//    caches while one is stale (bounded), and leaves t in LDS as two fp16 planes in fragment order; the wavefronts share
//    B's tiles.
//  - The ranges' accumulators are added through LDS in a fixed order.  With S > 1 the contraction is cut into S parts in
//    different workgroups, which write fp32 partial outputs that a second kernel adds in a fixed order.
//
// LDS slot of a chunk: 16-byte piece q of token row t sits at piece index 16 t + (q ^ (t & 15)).
#include "segments.hpp"

#include <type_traits>

namespace eora {

constexpr int WQ_NW = 8, WQ_NT = WQ_NW * 64;
constexpr size_t WQ_LDS_MAX = 160 * 1024 - 256;            // dynamic LDS of a workgroup at most

// the member's value of an argument array without a run-time index into kernel arguments
template <typename T>
__device__ __forceinline__ T wq_pick(const T (&v)[4], int m)
{
    T r = v[0];
    r = m == 1 ? v[1] : r;
    r = m == 2 ? v[2] : r;
    r = m == 3 ? v[3] : r;
    return r;
}

// where lane `lane` finds, for piece i of a chunk (token rows 4 i .. 4 i + 3), its 16 bytes of x: row offset in halves
__device__ __forceinline__ size_t wq_xrow(const WideArgs& a, int m0, int i, int lane)
{
    const int row = m0 + 4 * i + (lane >> 4);
    // rows beyond the tokens: all their lanes read one valid piece (their results are dropped)
    return row < a.M ? (size_t)row * a.d_in + 8 * (lane & 15) : (size_t)m0 * a.d_in;
}
__device__ __forceinline__ int wq_xdst(int i, int lane)
{
    const int t = 4 * i + (lane >> 4);
    return (t * 16 + ((lane & 15) ^ (t & 15))) * 16;
}
// fragment piece p (columns 8 p .. 8 p + 7 of the chunk) of token row n of a token block
__device__ __forceinline__ int wq_frag(int n, int p) { return (n * 16 + (p ^ n)) * 16; }

// ---- producer: one block of A, one range of the contraction, TB token blocks -------------------------------------------
// FEW: one to four tokens, the first 1 KiB piece of a chunk alone
template <int FA, int TB, bool FEW>
__device__ __forceinline__ void wq_produce(const WideArgs& a, const void* A, const _Float16* A_scales, int rho, int m0, int ka, int len,
                                           unsigned char* xs, int lane, f4 (&acc)[TB])
{
    constexpr int NT = 128 / Fmt<FA>::KT, NMF = Fmt<FA>::KT / 32, NP = FEW ? 1 : 4 * TB;
    const int n = lane & 15, j = lane >> 4;
    const Factor fa{(const uint32_t*)A, A_scales, a.d_in / Fmt<FA>::KT};
    const int last = a.d_in / 128 - 1;
    auto tile_at = [&](int s) {
        const int k = ka + (s < len ? s : (len > 0 ? len - 1 : 0));
        return k < last ? k : last;
    };
    FTile<FA> at[2][NT];
    u4 xr[NP];
    auto load_a = [&](FTile<FA> (&t)[NT], int s) {
        const int k = tile_at(s);
#pragma unroll
        for (int i = 0; i < NT; ++i) load_ftile<FA>(t[i], fa, rho, k * NT + i, lane);
    };
    auto load_x = [&](int s) {
        const _Float16* p = a.x + (size_t)tile_at(s) * 128;
#pragma unroll
        for (int i = 0; i < NP; ++i) xr[i] = *(const u4*)(p + wq_xrow(a, m0, i, lane));
    };
    load_x(0);
    load_a(at[0], 0);
    load_a(at[1], 1);
    for (int s0 = 0; s0 < len; s0 += 2) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int s = s0 + h;
            if (s < len) {
#pragma unroll
                for (int i = 0; i < NP; ++i) *(u4*)(xs + wq_xdst(i, lane)) = xr[i];
                load_x(s + 1);
                asm volatile("" ::: "memory");            // (the fragments read below were written by other lanes of this wavefront)
                if constexpr (FA == S_F16) {
#pragma unroll
                    for (int t = 0; t < NT; ++t) {
                        h8 b[1];
                        decode_tile<FA>(at[h][t].w, 8u, b);
#pragma unroll
                        for (int tb = 0; tb < TB; ++tb) acc[tb] = mfma16(*(const h8*)(xs + tb * 4096 + wq_frag(n, 4 * t + j)), b[0], acc[tb]);
                    }
                } else {
                    h8 b[NMF];
                    decode_tile<FA>(at[h][0].w, 8u, b);
                    const float sc = (float)at[h][0].sc;
#pragma unroll
                    for (int tb = 0; tb < TB; ++tb) {
                        f4 part = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                        for (int t = 0; t < NMF; ++t) part = mfma16(*(const h8*)(xs + tb * 4096 + wq_frag(n, 4 * j + t)), b[t], part);
                        acc[tb] += sc * part;
                    }
                }
                asm volatile("" ::: "memory");
                load_a(at[h], s + 2);
            }
        }
    }
}

// ---- consumer: acc += t.B^T for the wavefront's row blocks, its share of B's tiles -------------------------------------
// planes: t of TB token blocks as a high and a low fp16 part, piece p (columns 8 p ..) of token n of block tb at
// tb * tbs + p * 272 + 16 n; the low plane `plane` bytes behind
template <int FE, int RW>
__device__ __forceinline__ void wq_up_load(const Factor& fb, const int (&R)[RW], int g, int lane, uint32_t (&bw)[RW][4], _Float16 (&bs)[RW])
{
    constexpr int W = Fmt<FE>::WORDS;
    g = g < fb.ntk ? g : 0;                               // (a wavefront without a tile fetches a valid one)
#pragma unroll
    for (int rw = 0; rw < RW; ++rw) {
        FTile<FE> t;
        load_ftile<FE>(t, fb, R[rw], g, lane);
#pragma unroll
        for (int i = 0; i < W; ++i) bw[rw][i] = t.w[i];
        bs[rw] = t.sc;
    }
}

// tiles g0 + first, + STRIDE, ... < g1; have: the first one's words are in bw already
template <int FE, int TB, int RW, int STRIDE>
__device__ __forceinline__ void wq_up(const Factor& fb, const int (&R)[RW], int first, bool have, int tbs, int plane, int lane,
                                      uint32_t (&bw)[RW][4], _Float16 (&bs)[RW], int g0, int g1, f4 (&acc)[RW][TB])
{
    constexpr int KT = Fmt<FE>::KT, NMF = KT / 32, W = Fmt<FE>::WORDS;
    const int n = lane & 15, j = lane >> 4;
    for (int g = g0 + first; g < g1; g += STRIDE) {
        if (g != g0 + first || !have) wq_up_load<FE, RW>(fb, R, g, lane, bw, bs);
#pragma unroll
        for (int rw = 0; rw < RW; ++rw) {
            uint32_t w[W];
#pragma unroll
            for (int i = 0; i < W; ++i) w[i] = bw[rw][i];
            h8 b[NMF];
            decode_tile<FE>(w, 8u, b);
#pragma unroll
            for (int tb = 0; tb < TB; ++tb) {
                f4 part = {0.f, 0.f, 0.f, 0.f};
                if constexpr (FE == S_F16) part = acc[rw][tb];
#pragma unroll
                for (int q = 0; q < NMF; ++q) {
                    const unsigned char* p = eora_smem + tb * tbs + ((KT / 8) * (g - g0) + (KT / 32) * j + q) * 272 + 16 * n;
                    part = mfma16(*(const h8*)p, b[q], part);
                    part = mfma16(*(const h8*)(p + plane), b[q], part);
                }
                if constexpr (FE == S_F16) acc[rw][tb] = part;
                else acc[rw][tb] += (float)bs[rw] * part;
            }
        }
    }
}

// ONE_ORDER (one to four tokens): sums in an order that no split of the workgroup changes, so that a linear in a group's
// launch and alone has the same bits.  There are eight partial sums whatever NWK is, tile k of the backbone and of B going
// to number k modulo 8: a wavefront takes tiles wk, wk + NWK, ..., turn and turn about into its 8 / NWK accumulators.  They
// are added as ((0+4)+(2+6))+((1+5)+(3+7)).
template <int FM, int TB, int RW, int NWR, int NWK, bool LOWRANK, bool ONE_ORDER>
__global__ __launch_bounds__(WQ_NT, TB == 1 && (NWR > 1 || (ONE_ORDER && LOWRANK)) ? 4 : 2) void wide_q_kernel(WideArgs a)
{
    static_assert(NWR * NWK == WQ_NW, "eight wavefronts");
    static_assert(!ONE_ORDER || TB == 1, "one token block");
    constexpr int NV = ONE_ORDER ? 8 / NWK : 1;           // accumulators per wavefront and output tile
    constexpr int SLOT = TB * 4096;                       // bytes: 16 TB tokens x 128 columns
    constexpr int NSLOT = NWR == 1 ? 1 : 2;
    // 1 KiB pieces of a chunk (four token rows each) per wavefront.  With one to four tokens the first piece is all there is,
    // and the others' places in LDS keep whatever they hold: rows of a matrix product that nobody reads.  (Two row blocks
    // with 3-bit and 2-bit codes: one piece alone makes the compiler spill.)  The registers saved let two workgroups of one
    // row block share a compute unit: 14336 x 4096 W4, three tokens 20.3 -> 15.7 us, 1024 x 1024, one token 5.7 -> 5.2.
    constexpr int XN = ONE_ORDER && (NWR == 1 || FM == S_Q4) ? 1 : (4 * TB) / NWR;
    constexpr int PX = XN > 8 ? 1 : 2;                    // steps between a request for x and its LDS write
    // Two and more token blocks, wavefronts that share x through LDS: the next chunk's writes and the requests for the one behind it are
    // spread over the step (a compute unit takes in 64 bytes a cycle; all at once they hold a wavefront up for 270 .. 640 cycles
    // of 2900), fragments are read a quarter of a step ahead, and a wavefront's priority falls as it gets through the step (by
    // age alone the older of a SIMD's two runs ahead and waits at the barrier).  64 tokens, bare: 28672 x 4096 W4 30.6 -> 27.8 us,
    // 4096 x 4096 10.2 -> 9.5.  With one token block the writes come too late that way (14336 x 1152, ten tokens 6.4 -> 6.7).
    constexpr bool SPREAD = NWR > 1 && TB > 1;
    constexpr int D = RW >= 4 ? 2 : 4;                    // steps between a request for a stored tile and its use
    static_assert((4 * TB) % NWR == 0, "the pieces of a chunk divide evenly over a range's wavefronts");
    __shared__ uint32_t s_epoch;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 15, j = lane >> 4;
    const int bid = blockIdx.x;
    const int G = a.d_in / 128;
    const int ntg = a.ntg;

    uint32_t epoch_v = 0;
    if constexpr (LOWRANK) {
        if (tid == 0) epoch_v = ld_relaxed(&a.hdr[HDR_EPOCH]);
        if (bid < a.nprod) {
            // ===================================================================== producer
            __builtin_amdgcn_s_setprio(3);
            const int NRB = a.r / 16;
            int u = bid;
            const int rho = u % NRB; u /= NRB;
            const int kc = u % a.kcn; u /= a.kcn;
            const int tg = u % ntg, mem = u / ntg;
            const int m0 = tg * TB * 16;
            const int pa = G * kc / a.kcn, pb = G * (kc + 1) / a.kcn;
            const int ka = pa + (pb - pa) * wave / WQ_NW, kb = pa + (pb - pa) * (wave + 1) / WQ_NW;
            f4 acc[TB];
#pragma unroll
            for (int tb = 0; tb < TB; ++tb) acc[tb] = f4{0.f, 0.f, 0.f, 0.f};
            const void* A = wq_pick(a.A, mem);
            const _Float16* As = wq_pick(a.A_scales, mem);
            unsigned char* xs = eora_smem + wave * SLOT;
            if (a.fa == S_F16) wq_produce<S_F16, TB, ONE_ORDER>(a, A, As, rho, m0, ka, kb - ka, xs, lane, acc);
            else if (a.fa == S_Q4S128) wq_produce<S_Q4S128, TB, ONE_ORDER>(a, A, As, rho, m0, ka, kb - ka, xs, lane, acc);
            else wq_produce<S_Q3S128, TB, ONE_ORDER>(a, A, As, rho, m0, ka, kb - ka, xs, lane, acc);
            if (tid == 0) {
                s_epoch = epoch_v;
                arrive(epoch_v, a.hdr, bid);
            }
            __syncthreads();                              // x is dead: the partial tiles go over it
            f4* red = (f4*)eora_smem;                     // [wavefront][token block][lane]
#pragma unroll
            for (int tb = 0; tb < TB; ++tb) red[(wave * TB + tb) * 64 + lane] = acc[tb];
            __syncthreads();
            if (wave < TB) {
                const int tb = wave;
                f4 v = red[tb * 64 + lane];
#pragma unroll
                for (int w = 1; w < WQ_NW; ++w) v += red[(w * TB + tb) * 64 + lane];
                // [member][token group][kc][token][r] pairs, one write-through store each
                unsigned long long* dst = a.tpair + (((size_t)(mem * ntg + tg) * a.kcn + kc) * (16 * TB) + 16 * tb) * a.r + 16 * rho + n;
                const float vs[4] = {v.x, v.y, v.z, v.w};
                const unsigned long long tag = (unsigned long long)(s_epoch + 1) << 32;
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (m0 + 16 * tb + 4 * j + i < a.M)
                        __hip_atomic_store(&dst[(size_t)(4 * j + i) * a.r], tag | __builtin_bit_cast(uint32_t, vs[i]), __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT);
            }
            return;
        }
    }

    // ========================================================================= consumer
    const int wr = wave % NWR, wk = wave / NWR;
    int mem = 0;
#pragma unroll
    for (int i = 1; i < 4; ++i)
        if (i < a.n && bid >= a.first[i]) mem = i;
    const int RBs = wq_pick(a.d_out, mem) / 16;
    int rg = bid - wq_pick(a.first, mem), tg = 0, part_id = 0;
    if (a.S > 1 || ntg > 1) {
        // workgroups that read the same stored tiles (the token groups of one row group) sit eight apart: same XCD, same L2
        const int nrg = (RBs + NWR * RW - 1) / (NWR * RW);
        part_id = rg / (nrg * ntg);                       // which part of the contraction (S > 1)
        const int c = rg - part_id * nrg * ntg;
        const int oct = c / (8 * ntg), in_oct = c - oct * 8 * ntg;
        const int width = nrg - 8 * oct < 8 ? nrg - 8 * oct : 8;     // row groups of this octet
        tg = in_oct / width;
        rg = 8 * oct + in_oct - tg * width;
    }
    const int m0 = tg * TB * 16;
    const int ga0 = a.S > 1 ? G * part_id / a.S : 0, ga1 = a.S > 1 ? G * (part_id + 1) / a.S : G;         // this workgroup's tiles of a row block
    int R[RW];
#pragma unroll
    for (int rw = 0; rw < RW; ++rw) {
        const int Rw = rg * NWR * RW + wr * RW + rw;
        R[rw] = Rw < RBs ? Rw : RBs - 1;                  // a ragged last row group: computed on the last block, not stored
    }
    const uint32_t* const w = (const uint32_t*)wq_pick(a.w, mem);
    const _Float16* const w_scales = wq_pick(a.w_scales, mem);
    const uint32_t* const w_zeros = wq_pick(a.w_zeros, mem);
    const int gdiv = a.group / 128, NG = a.ng, NGW = (NG + 7) / 8;
    // quantisation group of tile k: k / gdiv by a multiplication and a correction, without a branch
    const uint32_t gmagic = a.gmagic;
    auto group_of = [&](int k) {
        const uint32_t q = (uint32_t)(((unsigned long long)(uint32_t)k * gmagic) >> 31);
        return (int)(q * (uint32_t)gdiv > (uint32_t)k ? q - 1 : q);
    };
    struct Pre { uint32_t w[Fmt<FM>::WORDS]; };
    Pre pre[D][RW];
    unsigned char* const xk = eora_smem + wk * NSLOT * SLOT;
    size_t xsrc[XN];
    int xdst[XN];
#pragma unroll
    for (int i = 0; i < XN; ++i) {
        xsrc[i] = wq_xrow(a, m0, wr + i * NWR, lane);
        xdst[i] = wq_xdst(wr + i * NWR, lane);
    }
    u4 xr[PX][XN];
    f4 accs[NV][RW][TB];
    f4 (&acc)[RW][TB] = accs[0];
#pragma unroll
    for (int v = 0; v < NV; ++v)
#pragma unroll
        for (int rw = 0; rw < RW; ++rw)
#pragma unroll
            for (int tb = 0; tb < TB; ++tb) accs[v][rw][tb] = f4{0.f, 0.f, 0.f, 0.f};
    int poff[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) poff[t] = wq_frag(n, 4 * j + t);
    // Group scales and zero-point words of the workgroup's rows sit in LDS behind the slots, [group][row] and
    // [word][row]: a scale is two bytes of a 64-byte row segment, and sixteen rows' worth of it per tile from global
    // memory is sixteen cache lines per tile (gate+up at 64 tokens, bare: 33.6 us that way, 32.5 this way).
    constexpr int ROWS = NWR * RW * 16;
    uint16_t* const m_sc = (uint16_t*)(eora_smem + NWK * NSLOT * SLOT);
    uint32_t* const m_zq = (uint32_t*)(m_sc + (size_t)ROWS * a.seg);

    // the contraction in segments of at most a.seg tiles (one for every usual shape): their scales fit the LDS
    for (int ga = ga0; ga < ga1; ga += a.seg) {
    const int gl = ga1 - ga < a.seg ? ga1 - ga : a.seg;
    // this range's tiles: consecutive ones, or (ONE_ORDER) every NWK-th
    const int ka = ONE_ORDER ? ga + wk : ga + gl * wk / NWK;
    const int len = ONE_ORDER ? (gl - wk + NWK - 1) / NWK : ga + gl * (wk + 1) / NWK - ka;       // (gl + NWK - 1 >= wk)
    constexpr int STRIDE = ONE_ORDER ? NWK : 1;
    const int steps = (gl + NWK - 1) / NWK;
    auto tile_at = [&](int s) {                           // tile (= chunk of x) of step s of this range
        const int k = ka + STRIDE * (s < len ? s : (len > 0 ? len - 1 : 0));
        return k < G - 1 ? k : G - 1;
    };
    auto load_tile = [&](Pre& p, int rw, int s) {
        load_words<Fmt<FM>::WORDS>(p.w, w + (((size_t)R[rw] * G + tile_at(s)) * 64 + lane) * Fmt<FM>::WORDS);
    };
    auto load_x = [&](u4 (&v)[XN], int s) {
        const _Float16* p = a.x + (size_t)tile_at(s) * 128;
#pragma unroll
        for (int i = 0; i < XN; ++i) v[i] = *(const u4*)(p + xsrc[i]);
    };
    const int g_lo = group_of(ga), ng = group_of(ga + gl - 1) - g_lo + 1, z_lo = g_lo >> 3, nz = ((g_lo + ng - 1) >> 3) - z_lo + 1;
    if (ga > ga0) __syncthreads();                        // the previous segment's slots and scales are dead
    // All requests of the start before the first wait, the scales' first (loads return in the order of their requests).
    // Thread -> row tid % ROWS, pieces from tid / ROWS on: no division, and consecutive threads write consecutive rows.
    constexpr int TPR = WQ_NT / ROWS;
    const int mrow = tid % ROWS, mq = tid / ROWS, mblk = rg * NWR * RW + (mrow >> 4);
    const size_t msrc = (size_t)(mblk < RBs ? mblk : RBs - 1) * 16 + (mrow & 15);       // a ragged last row group: the last block again
    const uint16_t* const ps = (const uint16_t*)w_scales + msrc * NG + g_lo;
    const uint32_t* const pz = w_zeros + msrc * NGW + z_lo;
    const bool by8 = ((NG | g_lo | ng) & 7) == 0;         // eight scales in one aligned 16-byte load
    u4 ms = {0u, 0u, 0u, 0u};
    if (by8) {
        ms = *(const u4*)(ps + (8 * mq < ng ? 8 * mq : 0));
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) ms[i] = ps[mq + i * TPR < ng ? mq + i * TPR : 0];
    }
    const uint32_t mz = pz[mq < nz ? mq : 0];
#pragma unroll
    for (int s = 0; s < PX; ++s) load_x(xr[s], s);
#pragma unroll
    for (int s = 0; s < D; ++s)
#pragma unroll
        for (int rw = 0; rw < RW; ++rw) load_tile(pre[s][rw], rw, s);
    if (by8) {
        if (8 * mq < ng) {
#pragma unroll
            for (int i = 0; i < 8; ++i) m_sc[(8 * mq + i) * ROWS + mrow] = (uint16_t)(ms[i >> 1] >> (16 * (i & 1)));
        }
        for (int g = 8 * (mq + TPR); g < ng; g += 8 * TPR) {
            const u4 v = *(const u4*)(ps + g);
#pragma unroll
            for (int i = 0; i < 8; ++i) m_sc[(g + i) * ROWS + mrow] = (uint16_t)(v[i >> 1] >> (16 * (i & 1)));
        }
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (mq + i * TPR < ng) m_sc[(mq + i * TPR) * ROWS + mrow] = (uint16_t)ms[i];
        for (int g = mq + 4 * TPR; g < ng; g += TPR) m_sc[g * ROWS + mrow] = ps[g];
    }
    if (mq < nz) m_zq[mq * ROWS + mrow] = mz;
    for (int z = mq + TPR; z < nz; z += TPR) m_zq[z * ROWS + mrow] = pz[z];
    if constexpr (LOWRANK) {
        if (tid == 0 && ga == ga0) {
            s_epoch = epoch_v;
            arrive(epoch_v, a.hdr, bid);
        }
    }
    if constexpr (NWR > 1) {                              // chunk 0 -> slot 0
#pragma unroll
        for (int i = 0; i < XN; ++i) *(u4*)(xk + xdst[i]) = xr[0][i];
        load_x(xr[0], PX);
    } else {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();                     // the scales are visible (NWR > 1: with the first chunk)
    }
    auto step = [&](auto itag, int s) {
        constexpr int i = decltype(itag)::value;          // s % D
        const unsigned char* xs = xk;
        if constexpr (NWR > 1) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");       // own LDS writes of chunk s done
            __builtin_amdgcn_s_barrier();                 // chunk s is visible, everyone has left the other slot
            xs = xk + (i & 1) * SLOT;
            if constexpr (!SPREAD) {
#pragma unroll
                for (int q = 0; q < XN; ++q) *(u4*)(xk + ((i + 1) & 1) * SLOT + xdst[q]) = xr[(i + 1) % PX][q];
                load_x(xr[(i + 1) % PX], s + 1 + PX);
            }
        } else {
#pragma unroll
            for (int q = 0; q < XN; ++q) *(u4*)(xk + xdst[q]) = xr[i % PX][q];
            load_x(xr[i % PX], s + PX);
        }
        asm volatile("" ::: "memory");                    // (fragments are read by other lanes than the ones that wrote them)
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (SPREAD) {
            // (a step past the range's end goes through the motions with a valid chunk and tile of the segment; nothing of it is added)
            f4 part[RW][TB];
            h8 b[2][RW], xf[2][TB];
            uint32_t z[RW];
            float sc[RW];
            const int grp = group_of(tile_at(s)), zs = 4 * (grp & 7);
            const int lrow = wr * RW * 16 + n;
#pragma unroll
            for (int rw = 0; rw < RW; ++rw) {
                sc[rw] = (float)__builtin_bit_cast(_Float16, m_sc[(grp - g_lo) * ROWS + lrow + 16 * rw]);
                z[rw] = m_zq[((grp >> 3) - z_lo) * ROWS + lrow + 16 * rw];
#pragma unroll
                for (int tb = 0; tb < TB; ++tb) part[rw][tb] = f4{0.f, 0.f, 0.f, 0.f};
            }
#pragma unroll
            for (int tb = 0; tb < TB; ++tb) xf[0][tb] = *(const h8*)(xs + tb * 4096 + poff[0]);
#pragma unroll
            for (int rw = 0; rw < RW; ++rw) {
                z[rw] = (z[rw] >> zs) & 0xFu;
                b[0][rw] = decode_frag<0>(pre[i][rw].w, z[rw]);
            }
            // quarter t: its MFMAs, and between them the decoding and the fragments of the next one and a share of x
            auto quarter = [&](auto ttag) __attribute__((always_inline)) {
                constexpr int t = decltype(ttag)::value;
                if constexpr (t < 3) {
#pragma unroll
                    for (int tb = 0; tb < TB; ++tb) xf[(t + 1) & 1][tb] = *(const h8*)(xs + tb * 4096 + poff[t + 1]);
                }
#pragma unroll
                for (int tb = 0; tb < TB; ++tb)
#pragma unroll
                    for (int rw = 0; rw < RW; ++rw) part[rw][tb] = mfma16(xf[t & 1][tb], b[t & 1][rw], part[rw][tb]);
                if constexpr (t < 3) {
#pragma unroll
                    for (int rw = 0; rw < RW; ++rw) b[(t + 1) & 1][rw] = decode_frag<t + 1>(pre[i][rw].w, z[rw]);
                }
#pragma unroll
                for (int q = XN * t / 4; q < XN * (t + 1) / 4; ++q) {
                    *(u4*)(xk + ((i + 1) & 1) * SLOT + xdst[q]) = xr[(i + 1) % PX][q];
                    xr[(i + 1) % PX][q] = *(const u4*)(a.x + (size_t)tile_at(s + 1 + PX) * 128 + xsrc[q]);
                }
                __builtin_amdgcn_sched_barrier(0);
            };
            __builtin_amdgcn_s_setprio(3);
            quarter(std::integral_constant<int, 0>{});
            __builtin_amdgcn_s_setprio(2);
            quarter(std::integral_constant<int, 1>{});
            __builtin_amdgcn_s_setprio(1);
            quarter(std::integral_constant<int, 2>{});
            __builtin_amdgcn_s_setprio(0);
            quarter(std::integral_constant<int, 3>{});
            if (s < len) {                                // uniform over the wavefront; no global load inside
#pragma unroll
                for (int rw = 0; rw < RW; ++rw) {
#pragma unroll
                    for (int tb = 0; tb < TB; ++tb) accs[i % NV][rw][tb] += sc[rw] * part[rw][tb];
                }
            }
        } else if (s < len) {                             // uniform over the wavefront; no global load inside
            h8 b[RW][4];
            f4 part[RW][TB];
            const int grp = group_of(ka + STRIDE * s), zs = 4 * (grp & 7);
            const int lrow = wr * RW * 16 + n;
            float sc[RW];
#pragma unroll
            for (int rw = 0; rw < RW; ++rw) {
                sc[rw] = (float)__builtin_bit_cast(_Float16, m_sc[(grp - g_lo) * ROWS + lrow + 16 * rw]);
                decode_tile<FM>(pre[i][rw].w, (m_zq[((grp >> 3) - z_lo) * ROWS + lrow + 16 * rw] >> zs) & 0xFu, b[rw]);
#pragma unroll
                for (int tb = 0; tb < TB; ++tb) part[rw][tb] = f4{0.f, 0.f, 0.f, 0.f};
            }
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int tb = 0; tb < TB; ++tb) {
                    const h8 xf = *(const h8*)(xs + tb * 4096 + poff[t]);
#pragma unroll
                    for (int rw = 0; rw < RW; ++rw) part[rw][tb] = mfma16(xf, b[rw][t], part[rw][tb]);
                }
#pragma unroll
            for (int rw = 0; rw < RW; ++rw) {
#pragma unroll
                for (int tb = 0; tb < TB; ++tb) accs[i % NV][rw][tb] += sc[rw] * part[rw][tb];
            }
        }
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int rw = 0; rw < RW; ++rw) load_tile(pre[i][rw], rw, s + D);
        __builtin_amdgcn_sched_barrier(0);
    };
    // D steps at a time without a branch around a load, so that the compiler knows how many requests follow the one it
    // waits for (with a test per step it waits for all of them); the last up to D - 1 apart
    int s0 = 0;
    for (; s0 + D <= steps; s0 += D) {
        step(std::integral_constant<int, 0>{}, s0);
        step(std::integral_constant<int, 1>{}, s0 + 1);
        if constexpr (D == 4) {
            step(std::integral_constant<int, 2>{}, s0 + 2);
            step(std::integral_constant<int, 3>{}, s0 + 3);
        }
    }
    if (s0 < steps) step(std::integral_constant<int, 0>{}, s0);
    if constexpr (D == 4) {
        if (s0 + 1 < steps) step(std::integral_constant<int, 1>{}, s0 + 1);
        if (s0 + 2 < steps) step(std::integral_constant<int, 2>{}, s0 + 2);
    }
    }
    __syncthreads();                                      // nobody reads x any more: the LDS is reused below

    // ---- low-rank continuation: acc[token][row] += t[token][:] . B[row][:] ----------------------------------
    if constexpr (LOWRANK) {
        // with S > 1 every part takes its share [g0, g1) of B's tiles (and reads those columns of t only)
        const int KTb = a.fe == S_F16 ? 32 : a.fe == S_Q4S64 ? 64 : 128, ntk = a.r / KTb;
        const int g0 = a.S > 1 ? ntk * part_id / a.S : 0, g1 = a.S > 1 ? ntk * (part_id + 1) / a.S : ntk;
        if (g0 < g1) {                                    // (uniform over the workgroup)
            if (a.spin_limit < 0) {                       // test hook: every wait counts as expired
                if (tid == 0) atomicOr(&a.hdr[HDR_ERROR], 1u);
            } else {
                const int P = (g1 - g0) * KTb / 8, tbs = P * 272, plane = TB * tbs;
                const uint32_t want = s_epoch + 1;
                // the first tiles of B on their way before t is read (their words do not depend on it)
                const Factor fb{(const uint32_t*)wq_pick(a.B, mem), wq_pick(a.B_scales, mem), ntk};
                uint32_t bw[RW][4];
                _Float16 bs[RW];
                if (a.fe == S_F16) wq_up_load<S_F16, RW>(fb, R, g0 + wk, lane, bw, bs);
                else if (a.fe == S_Q4S128) wq_up_load<S_Q4S128, RW>(fb, R, g0 + wk, lane, bw, bs);
                else if (a.fe == S_Q4S64) wq_up_load<S_Q4S64, RW>(fb, R, g0 + wk, lane, bw, bs);
                else wq_up_load<S_Q3S128, RW>(fb, R, g0 + wk, lane, bw, bs);
                const int rows = a.M - m0 < 16 * TB ? a.M - m0 : 16 * TB;
                const unsigned long long* const src = a.tpair + (size_t)(mem * ntg + tg) * a.kcn * (16 * TB) * a.r + g0 * KTb;
                bool good_all = true;
                for (int e = tid; e < rows * P; e += WQ_NT) {
                    const int tok = e / P, p = e - tok * P;
                    const unsigned long long* const q = src + (size_t)tok * a.r + 8 * p;
                    float v[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
                    uint32_t bad = 0;
#pragma unroll 2
                    for (int kc = 0; kc < a.kcn; ++kc) {  // fixed order; ordinary cached loads, the tags say whether they were late enough
                        const u4* pk = (const u4*)(q + (size_t)kc * (16 * TB) * a.r);
#pragma unroll
                        for (int h = 0; h < 4; ++h) {
                            const u4 pr = pk[h];
                            const uint32_t e0 = pr[0], t0 = pr[1], e1 = pr[2], t1 = pr[3];
                            bad |= (t0 ^ want) | (t1 ^ want);
                            v[2 * h] += __builtin_bit_cast(float, e0);
                            v[2 * h + 1] += __builtin_bit_cast(float, e1);
                        }
                    }
                    for (int spins = 0; bad != 0 && spins <= a.spin_limit; ++spins) {
                        bad = 0;
#pragma unroll
                        for (int h = 0; h < 8; ++h) v[h] = 0.f;
                        for (int kc = 0; kc < a.kcn; ++kc)
#pragma unroll
                            for (int h = 0; h < 8; ++h) {
                                const unsigned long long pr = __hip_atomic_load(q + (size_t)kc * (16 * TB) * a.r + h, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                                bad |= (uint32_t)(pr >> 32) ^ want;
                                v[h] += __builtin_bit_cast(float, (uint32_t)pr);
                            }
                    }
                    good_all = good_all && bad == 0;
                    // several adapters side by side: a token row keeps its own adapter's columns (r_per is a multiple of 8)
                    const bool keep = !a.adapter || a.adapter[m0 + tok] == (g0 * KTb + 8 * p) / a.r_per;
                    h8 hi, lo;
#pragma unroll
                    for (int h = 0; h < 8; ++h) {
                        const float t = keep ? v[h] : 0.f;
                        hi[h] = (_Float16)t;
                        lo[h] = (_Float16)(t - (float)hi[h]);
                    }
                    unsigned char* const d = eora_smem + (tok >> 4) * tbs + p * 272 + 16 * (tok & 15);
                    *(h8*)d = hi;
                    *(h8*)(d + plane) = lo;
                }
                if (!good_all) atomicOr(&a.hdr[HDR_ERROR], 1u);       // never expected: producers do not wait
                __syncthreads();
                auto up = [&](auto fmt) {
                    constexpr int FE = decltype(fmt)::value;
#pragma unroll
                    for (int v = 0; v < NV; ++v)          // (every NWK-th tile is this wavefront's)
                        wq_up<FE, TB, RW, NV * NWK>(fb, R, wk + NWK * v, v == 0, tbs, plane, lane, bw, bs, g0, g1, accs[v]);
                };
                if (a.fe == S_F16) up(std::integral_constant<int, S_F16>{});
                else if (a.fe == S_Q4S128) up(std::integral_constant<int, S_Q4S128>{});
                else if (a.fe == S_Q4S64) up(std::integral_constant<int, S_Q4S64>{});
                else up(std::integral_constant<int, S_Q3S128>{});
                __syncthreads();                          // t has been used: the LDS is reused below
            }
        }
    }

    // ---- add the ranges' accumulators in a fixed order, convert, store ---------------------------------------
    if constexpr (NV > 1) {
#pragma unroll
        for (int rw = 0; rw < RW; ++rw)
            acc[rw][0] = NV == 2 ? accs[0][rw][0] + accs[NV / 2][rw][0] : (accs[0][rw][0] + accs[NV / 2][rw][0]) + (accs[1][rw][0] + accs[NV - 1][rw][0]);
    }
    // through LDS as [range][token][row], so that a thread adds and stores eight consecutive rows of a token (rows of
    // 4 bytes more than a multiple of 16 banks keep the four token rows of a store apart)
    constexpr int RS = ROWS + 4;
    float* const red = (float*)eora_smem;
#pragma unroll
    for (int rw = 0; rw < RW; ++rw)
#pragma unroll
        for (int tb = 0; tb < TB; ++tb) {
            // register i is token row 4 j + i of the token block, output column n of the row block
            float* const d = red + ((size_t)wk * 16 * TB + 16 * tb + 4 * j) * RS + (wr * RW + rw) * 16 + n;
            const f4 v = acc[rw][tb];
            d[0] = v.x;
            d[RS] = v.y;
            d[2 * RS] = v.z;
            d[3 * RS] = v.w;
        }
    __syncthreads();
    _Float16* const y = wq_pick(a.y, mem);
    const int d_out = RBs * 16;
    for (int e = tid; e < 16 * TB * ROWS / 8; e += WQ_NT) {
        const int tok = e / (ROWS / 8), r8 = 8 * (e % (ROWS / 8));
        const int m = m0 + tok, o = rg * ROWS + r8;
        if (m >= a.M || o >= d_out) continue;
        const float* p = red + (size_t)tok * RS + r8;
        f4 v0, v1;
        if constexpr (ONE_ORDER) {
            f4 sums[2][NWK];
#pragma unroll
            for (int k2 = 0; k2 < NWK; ++k2) {
                sums[0][k2] = *(const f4*)(p + (size_t)k2 * 16 * RS);
                sums[1][k2] = *(const f4*)(p + (size_t)k2 * 16 * RS + 4);
            }
#pragma unroll
            for (int w2 = NWK / 2; w2 > 0; w2 /= 2)       // halves apart
#pragma unroll
                for (int k2 = 0; k2 < w2; ++k2) {
                    sums[0][k2] += sums[0][k2 + w2];
                    sums[1][k2] += sums[1][k2 + w2];
                }
            v0 = sums[0][0];
            v1 = sums[1][0];
        } else {
            v0 = *(const f4*)p;
            v1 = *(const f4*)(p + 4);
#pragma unroll
            for (int k2 = 1; k2 < NWK; ++k2) {
                v0 += *(const f4*)(p + (size_t)k2 * 16 * TB * RS);
                v1 += *(const f4*)(p + (size_t)k2 * 16 * TB * RS + 4);
            }
        }
        if (a.S > 1) {
            float* const q = a.ypart + (size_t)a.S * a.M * wq_pick(a.ycol, mem) + ((size_t)part_id * a.M + m) * d_out + o;
            *(f4*)q = v0;
            *(f4*)(q + 4) = v1;
        } else {
            *(h8*)(y + (size_t)m * d_out + o) = h8{(_Float16)v0[0], (_Float16)v0[1], (_Float16)v0[2], (_Float16)v0[3],
                                                   (_Float16)v1[0], (_Float16)v1[1], (_Float16)v1[2], (_Float16)v1[3]};
        }
    }
    if constexpr (LOWRANK) {
        if (bid == (int)gridDim.x - 1 && wave == WQ_NW - 1) {
            if (!advance_epoch(s_epoch, a.hdr, gridDim.x, lane, a.spin_limit) && lane == 0) atomicOr(&a.hdr[HDR_ERROR], 1u);
        }
    }
}

// ------------------------------------------------------------------------------------------------
// y = fp16(sum over the S parts, in order); one launch for all members
__global__ __launch_bounds__(256) void wide_q_sum_kernel(WideArgs a)
{
    int mem = 0, b = blockIdx.x;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const int nb = (int)(((size_t)a.M * a.d_out[i] / 8 + 255) / 256);
        if (mem == i && i + 1 < a.n && b >= nb) {
            b -= nb;
            mem = i + 1;
        }
    }
    const size_t count = (size_t)a.M * wq_pick(a.d_out, mem);
    const size_t e = 8 * ((size_t)b * 256 + threadIdx.x);
    if (e >= count) return;
    const float* p = a.ypart + (size_t)a.S * a.M * wq_pick(a.ycol, mem) + e;
    f4 v0 = *(const f4*)p, v1 = *(const f4*)(p + 4);
    for (int s = 1; s < a.S; ++s) {
        v0 += *(const f4*)(p + s * count);
        v1 += *(const f4*)(p + s * count + 4);
    }
    *(h8*)(wq_pick(a.y, mem) + e) = h8{(_Float16)v0[0], (_Float16)v0[1], (_Float16)v0[2], (_Float16)v0[3],
                                       (_Float16)v1[0], (_Float16)v1[1], (_Float16)v1[2], (_Float16)v1[3]};
}

// ------------------------------------------------------------------------------------------------
template <int FM, int TB, int RW, int NWR, int NWK, bool LOWRANK, bool ONE_ORDER>
static hipError_t launch_wide_one(WideArgs a, hipStream_t stream)
{
    constexpr int NSLOT = NWR == 1 ? 1 : 2;
    constexpr int ROWS = NWR * RW * 16;
    const size_t slots = (size_t)NWK * NSLOT * TB * 4096;
    // tiles whose scales (2 bytes a row) and zero-point words (4 bytes a row and eight groups, one more at either end) fit
    const int G = a.d_in / 128, gdiv = a.group / 128;
    size_t fit = (WQ_LDS_MAX - slots) / ROWS;
    fit = fit > 16 ? (fit - 16) * 2 / 5 : 0;
    if (fit < 8) return hipErrorInvalidValue;
    a.seg = (int)(fit < (size_t)G ? fit & ~(size_t)7 : G);
    size_t lds = slots + (size_t)ROWS * a.seg * 2 + (size_t)ROWS * (a.seg / 8 + 2) * 4;
    a.ng = G / gdiv;
    a.gmagic = (uint32_t)((0x80000000ull + gdiv - 1) / gdiv);
    const size_t red = (size_t)NWK * 16 * TB * (ROWS + 4) * 4, prod = (size_t)WQ_NW * TB * 4096, t = (size_t)2 * TB * (a.r / 8) * 272;
    lds = lds > red ? lds : red;
    if (LOWRANK) lds = lds > prod ? lds : prod;
    if (LOWRANK) lds = lds > t ? lds : t;
    auto kern = wide_q_kernel<FM, TB, RW, NWR, NWK, LOWRANK, ONE_ORDER>;
    if (lds > 48 * 1024) {
        hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    int total = a.nprod;
    for (int i = 0; i < 4; ++i) {
        a.first[i] = total;
        a.ycol[i] = i > 0 && i < a.n ? a.ycol[i - 1] + a.d_out[i - 1] : 0;
        if (i < a.n) total += (a.d_out[i] / 16 + NWR * RW - 1) / (NWR * RW) * a.ntg * a.S;
    }
    const int part_tiles = (G + a.S - 1) / a.S, segments = (part_tiles + a.seg - 1) / a.seg;         // of the longest part
    if (a.S == 1 && segments == 1) note_launch("wide_q FM=%d FA=%d NWR=%d NWK=%d TB=%d n=%d", FM, a.fa, NWR, NWK, TB, a.n);
    else note_launch("wide_q FM=%d FA=%d NWR=%d NWK=%d TB=%d parts=%d segments=%d n=%d", FM, a.fa, NWR, NWK, TB, a.S, segments, a.n);
    hipLaunchKernelGGL(kern, dim3(total), dim3(WQ_NT), lds, stream, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || a.S == 1) return e;
    int blocks = 0;
    for (int i = 0; i < a.n; ++i) blocks += (int)(((size_t)a.M * a.d_out[i] / 8 + 255) / 256);
    hipLaunchKernelGGL(wide_q_sum_kernel, dim3(blocks), dim3(256), 0, stream, a);
    return hipGetLastError();
}

template <int FM, int TB, bool LOWRANK, bool ONE_ORDER = false>
static hipError_t launch_wide_cfg(const WideArgs& a, int cfg, hipStream_t stream)
{
    if constexpr (!ONE_ORDER) {                           // (its eight row blocks' eighths do not fit 128 registers)
        if (cfg == 0) return launch_wide_one<FM, TB, 2, 4, 2, LOWRANK, false>(a, stream);
    }
    switch (cfg) {
        case 1: return launch_wide_one<FM, TB, 1, 4, 2, LOWRANK, ONE_ORDER>(a, stream);
        case 2: return launch_wide_one<FM, TB, 1, 2, 4, LOWRANK, ONE_ORDER>(a, stream);
        case 3: return launch_wide_one<FM, TB, 1, 1, 8, LOWRANK, ONE_ORDER>(a, stream);
        default: return hipErrorInvalidValue;
    }
}

// The split of a launch: token blocks of a workgroup, its row blocks and ranges (configuration 0..3), parts of the contraction
struct WidePlan { int tb, cfg, S; };
constexpr int ONE_ORDER_D_IN = 256 * 128;                  // longest contraction of the kernel that takes all sums in one order

// k-ranges of t: a producer's eight wavefronts take four chunks each (one range at d_in 4096: with two the consumers of a
// gate+up launch at 64 tokens lose more to the producers' compute units than t arrives earlier, 33.3 -> 37.4 us)
static int wide_kcn(const WideArgs& a, int tb)
{
    const int G = a.d_in / 128, ntg = ((a.M + 15) / 16 + tb - 1) / tb;
    int kcn = (G + 31) / 32;
    while (kcn > 1 && (size_t)a.n * ntg * tb * 16 * kcn * a.r > a.tpair_count) --kcn;
    return kcn;
}

static WidePlan wide_plan(const WideArgs& a)
{
    // The cheapest by steps.  A step of 128 columns per range costs STEP microseconds whatever the launch's size (LDS
    // traffic and the barrier), a workgroup's start, hand-over of t and end about 9; workgroups beyond the chip's slots come
    // in further rounds.  The sum of the parts: with three or four token blocks it grows with the parts and the output
    // (fitted with four at 41 and 64 tokens, two to eight parts; against 8 microseconds whatever the size: 64 x 14336 x 4096 W4
    // 27.4 -> 27.5 us, 80 x 11008 x 4096 bare 26.0); with one or two the fit splits too much (24 x 14336 x 4096
    // 21.4 -> 22.7) and 8 stays.  Measured on one-linear launches of 64 and 24 tokens, contractions of 4096 .. 14336 (down
    // projection of the 8B layer, 64 tokens: two row blocks per workgroup and one part 46.9 us, eight and seven parts 27.3).
    static const int per[4] = {8, 4, 2, 1}, ranges[4] = {2, 2, 4, 8};
    static const float STEP[4][4] = {{0.5f, 0.4f, 0.45f, 0.6f}, {0.85f, 0.55f, 0.65f, 1.2f}, {0.95f, 0.7f, 1.f, 2.f}, {1.2f, 0.85f, 1.3f, 2.8f}};
    const int yblocks = (a.M + 15) / 16, G = a.d_in / 128;
    size_t rows = 0;
    for (int i = 0; i < a.n; ++i) rows += a.d_out[i];
    auto workgroups = [&](int tb, int c, int S) {
        const int ntg = (yblocks + tb - 1) / tb;
        int cons = 0;
        for (int i = 0; i < a.n; ++i) cons += (a.d_out[i] / 16 + per[c] - 1) / per[c] * ntg;
        return cons * S + (a.r > 0 ? a.n * (a.r / 16) * wide_kcn(a, tb) * ntg : 0);
    };
    // Three token blocks where they make as many groups as four would (33..48, 65..96, 129..144 tokens): a step's requests for x,
    // fragments and MFMAs are a quarter fewer.  40 x 4096 x 2 x 14336 W4, rank 128: 29.2 -> 27.0 us; 48 x 8192 x 28672 W3 49.8 -> 44.9;
    // 96 x 8192 x 8192 W3 46.5 -> 41.0; 70 tokens, q+k+v of 4096, W2 24.5 -> 21.4.  Contractions beyond 32768 were not measured and keep
    // four.  Their steps and the 3 and 0.3 us of a sum of parts are fitted over 520 launches (20 shapes, 33 to 144 tokens, W4 and W3, ranks 0, 64
    // and 128), every split of each timed: 1.4 % above the best split on average, none 3 % above the split of four blocks.  (A step of 1 for eight row blocks, 2.5
    // and 0.5: 1.7 %; 48 x 14336 x 4096 W4, rank 128, 24.2 us in three parts of four row blocks, 22.3 with four token blocks, 21.8 in seven of eight.)
    const bool three = G <= 256 && (yblocks + 2) / 3 == (yblocks + 3) / 4;
    WidePlan best{yblocks < 3 ? yblocks : three ? 3 : 4, 0, 1};
    const int tb = best.tb;
    const float* const step_us = STEP[tb - 1];
    const float sum0 = tb == 4 ? 1.f : tb == 3 ? 3.f : 8.f, sum_part = tb >= 3 ? (tb == 4 ? 0.5f : 0.3f) + 4.2e-6f * (float)a.M * (float)rows : 0.f;
    float best_us = 1e30f;
    for (int c = a.M <= 4 ? 1 : 0; c < 4; ++c) {
        // workgroups the chip holds (registers)
        const int slots = tb == 1 && (c < 3 || (a.M <= 4 && a.r > 0 && a.d_in <= ONE_ORDER_D_IN)) ? 512 : 256;
        for (int S = 1; S <= 8; ++S) {
            // (one to four tokens stay whole: the parts would depend on the rows, and with them the order of the sums)
            if (S > 1 && (a.M <= 4 || S * ranges[c] > G || (size_t)S * a.M * rows > a.ypart_count)) break;
            const int rounds = (workgroups(tb, c, S) + slots - 1) / slots, tiles = (G + S - 1) / S;
            const float t = rounds * (9.f + step_us[c] * ((tiles + ranges[c] - 1) / ranges[c])) + (S > 1 ? sum0 + sum_part * S : 0.f);
            if (t < best_us) {
                best_us = t;
                best = WidePlan{tb, c, S};
            }
        }
    }
    // Small launches: fewer token blocks per workgroup, each group of them with workgroups of its own that read the same
    // stored tiles (from L2), where the whole launch then still has one workgroup per compute unit or less and at most
    // sixteen steps.  A step with one token block is a third as long as with four and the tiles are not what bounds such a
    // launch (33 x 4096 x 1024 W4, rank 64: four token blocks 15.5 us, two 10.0, one 8.0; 64 x 4096 x 4096 W4, 4-bit
    // factors: 18.8, 15.8, 15.8; 24 x 4096 x 1024 W3 bare: two 8.3, one 7.0; 48 x 2688 x 2688 W4 bare: 11.2, 8.3, 7.2).
    // With more steps or a second round the tiles' second reading and decoding shows (100 x 7296 x 2688 W3 bare: four
    // token blocks in three parts 18.6 us, two 22.1; 33 x 4096 x 11008 W4: 21.3, one 25.6), and with eight row blocks per
    // workgroup it is no gain (48 x 4096 x 14336 W3: 23.0, two 23.8).  Fixed costs and steps in microseconds from 172
    // shapes of 3 .. 256 tokens, every split of each timed: on average 0.89 of the time of the splits above, none slower.
    static const float FIXED[2] = {4.5f, 5.5f}, LOW_RANK = 1.8f;
    static const float BARE_LESS = 2.5f, TWO_LESS = 2.f;  // what the 9 above has too much without a low-rank term, with two token blocks
    static const float SMALL_STEP[2][4] = {{0.f, 0.5f, 0.55f, 0.6f}, {0.f, 0.5f, 0.8f, 1.2f}};
    if (a.r == 0) best_us -= BARE_LESS;
    if (tb == 2) best_us -= TWO_LESS;
    for (int t = 1; t < tb; t *= 2)
        for (int c = 1; c < 4; ++c) {
            const int steps = (G + ranges[c] - 1) / ranges[c];
            if (steps > 16 || workgroups(t, c, 1) > 256) continue;
            const float us = FIXED[t - 1] + (a.r > 0 ? LOW_RANK : 0.f) + SMALL_STEP[t - 1][c] * steps;
            if (us < best_us) {
                best_us = us;
                best = WidePlan{t, c, 1};
            }
        }
    return best;
}

// One to four tokens: every split takes the sums in one order (ONE_ORDER above), so that a group's results are those of
// separate calls bit for bit.  That needs scales in one segment in every split (the largest workgroup holds those of 296
// tiles) and, in a group, t in as many ranges as a member alone has them.
static bool wide_one_order(const WideArgs& a) { return a.M <= 4 && a.S == 1 && a.d_in <= ONE_ORDER_D_IN; }

bool wide_q_shares_launch(const WideArgs& a)
{
    if (a.n == 1 || a.M > 4) return true;
    WideArgs one = a;
    one.n = 1;
    return a.d_in <= ONE_ORDER_D_IN && wide_kcn(a, 1) == wide_kcn(one, 1);
}

template <int FM>
static hipError_t launch_wide_fm(WideArgs a, hipStream_t stream)
{
    const WidePlan p = wide_plan(a);
    a.ntg = ((a.M + 15) / 16 + p.tb - 1) / p.tb;
    a.kcn = wide_kcn(a, p.tb);
    a.nprod = a.r > 0 ? a.n * (a.r / 16) * a.kcn * a.ntg : 0;
    a.S = p.S;
    if (wide_one_order(a)) return a.r > 0 ? launch_wide_cfg<FM, 1, true, true>(a, p.cfg, stream) : launch_wide_cfg<FM, 1, false, true>(a, p.cfg, stream);
    if (a.r > 0) {
        switch (p.tb) {
            case 1: return launch_wide_cfg<FM, 1, true>(a, p.cfg, stream);
            case 2: return launch_wide_cfg<FM, 2, true>(a, p.cfg, stream);
            case 3: return launch_wide_cfg<FM, 3, true>(a, p.cfg, stream);
            default: return launch_wide_cfg<FM, 4, true>(a, p.cfg, stream);
        }
    }
    switch (p.tb) {
        case 1: return launch_wide_cfg<FM, 1, false>(a, p.cfg, stream);
        case 2: return launch_wide_cfg<FM, 2, false>(a, p.cfg, stream);
        case 3: return launch_wide_cfg<FM, 3, false>(a, p.cfg, stream);
        default: return launch_wide_cfg<FM, 4, false>(a, p.cfg, stream);
    }
}

hipError_t launch_wide_q(const WideArgs& a, int fm, hipStream_t stream)
{
    switch (fm) {
        case S_Q4: return launch_wide_fm<S_Q4>(a, stream);
        case S_Q3: return launch_wide_fm<S_Q3>(a, stream);
        case S_Q2: return launch_wide_fm<S_Q2>(a, stream);
        default: return hipErrorInvalidValue;
    }
}

// every word 0, except the epoch word, which starts at `epoch0`
__global__ void clear_words_kernel(uint32_t* p, int nwords, uint32_t epoch0)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < nwords) p[i] = i == HDR_EPOCH ? epoch0 : 0u;
}

hipError_t launch_clear_words(uint32_t* p, int nwords, uint32_t epoch0, hipStream_t stream)
{
    hipLaunchKernelGGL(clear_words_kernel, dim3((nwords + 255) / 256), dim3(256), 0, stream, p, nwords, epoch0);
    return hipGetLastError();
}

}  // namespace eora
