// Prefill (many tokens): y = x.What^T + t.B^T as ONE MFMA-bound GEMM whose contraction runs over
// d_in (backbone, dequantised on the way) and then over r (B's tiles with t = x.A^T as the
// activation) into the same fp32 accumulators (Sec. 3 forward equation, Alg. 1 step 7; the fusion of
// B's product into the backbone's output follows Sec. 4.5 / App. A.6).  t itself is a first, small
// launch with A as the weight operand (fp16 M x r into scratch): recomputing it per output tile would
// cost r / 128 times the backbone's MFMA work.  That launch, and launches of few output tiles, take the
// kernel of prefill128.hip; this one has 128, 192 or 256 tokens per workgroup.
//
// Workgroup: 8 wavefronts (2 along the tokens x 4 along the rows), tile = 64 TM tokens x 256 rows, contraction in steps of 64
// columns; a wavefront owns 32 TM tokens x 64 rows as blocks of v_mfma_f32_16x16x32_f16 (A: 16 rows of weights, B: 16 tokens;
// lane l holds columns 8 (l / 16) .. + 7 of row / token l % 16, result register v is row 4 (l / 16) + v of token l % 16).
//
// What bounds it is the card's power: with all compute units busy the clock falls to 1.3 .. 1.8 GHz, and the time follows the
// energy of the work more than its cycles.  Register-only loops over normally distributed activations and dequantised weights
// run at 2.02 PFLOP/s with 16x16x32 and at 1.75 with 32x32x16 (with zeros both reach 2.4), so the smaller form is taken; the
// library's GEMM reaches 1.47 on fp16 weights of the size below.  8192 tokens x 28672 rows, d_in 4096, 4 bits: 1466 us
// (1.31 PFLOP/s); the kernel before this one (128 x 256 tiles, 32x32x16, weights decoded into the registers of each
// wavefront, x read from LDS once per 32 rows) 1850 us.
//   - 256 tokens (TM = 4) share the decoding of a weight and the reading of x by 256 rows: 1926, 1652, 1466 us with 128, 192
//     and 256.  More does not fit: 128 accumulator registers of 256, and three slabs of x next to two of weights in LDS.
//   - Weights: every lane decodes 32 of them a step (one stored lane's words; exact integers code - zero, times the fp16 scale
//     of the group: one rounding, relative error <= 2^-11 per weight) and writes them to LDS as four 16-byte chunks, between
//     the MFMAs of the step before; the words are requested two steps ahead.
//   - x goes from memory to LDS without passing registers, one step ahead (through registers and ds_write: 1600 us).
//   - Both slabs are rows of 64 columns with the 16-byte chunks of a row XOR-ed by half the row's number: taking it that
//     accesses of 16 bytes per lane are served in groups of 16 lanes {0-3, 12-15, 20-23, 24-27}, ..., none has two lanes on a
//     bank.  The counters do not bear that out whole: 21 % of the LDS cycles are conflicts (2048 tokens, 256 a tile), of
//     which accesses is not known.
//   - A step has one barrier.  The last quarter of its MFMAs is carried out behind it, under the first LDS reads of the next.
//   - Requests for x are spread over the step (all at once, every wavefront waits for 350 cycles to get rid of them: 1572 us
//     instead of 1542), and a wavefront's priority falls as it gets through the step: left to age, wavefronts 0..3 run ahead
//     of those they share a SIMD with and idle for a third of the step at the barrier (1502 us instead of 1466).
//   - Scales come eight groups at a time (16 bytes per row): one by one their lines cost as many bytes of L2 as x does.
#include "segments.hpp"

namespace eora {


constexpr int PF_BN = 256;                            // output rows per workgroup
constexpr int PF_NW = 8, PF_NT = PF_NW * 64;          // wavefronts: 2 along the tokens x 4 along the rows
constexpr int PF_WS = PF_BN * 128;                    // one slab of weights: 256 rows x 64 columns fp16
constexpr int pf_bm(int tm) { return 64 * tm; }       // tokens per workgroup: TM blocks of 32 per wavefront
constexpr int pf_lds(int tm) { return 3 * pf_bm(tm) * 128 + 2 * PF_WS; }      // three slabs of x, two of weights

#define PF_SCHED() __builtin_amdgcn_sched_barrier(0)
// A slab in LDS is rows of 64 columns (128 bytes); the 16-byte chunk c of row R sits at slot c ^ ((R >> 1) & 7).
__device__ __forceinline__ int pf_slot(int row, int c) { return row * 128 + ((c ^ ((row >> 1) & 7)) << 4); }

// Scales and zero-points of the lane's row: those of eight consecutive groups where a row's allow 16-byte loads, else of one.
struct WScale {
    uint32_t s[4], z;
};

// Loads whose address is a uniform base and a 32-bit offset per lane: buffer instructions take both as they are (with plain
// pointers the compiler keeps 64-bit addresses per lane, and the kernel does not fit its registers).  The offsets are
// clamped to valid rows by the caller; the descriptor checks nothing.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t pf_rsrc(const void* p)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, -1, 0x00027000);
}

template <int WORDS>
__device__ __forceinline__ void pf_load(uint32_t (&w)[WORDS], __amdgpu_buffer_rsrc_t r, uint32_t lane_off, uint32_t off)
{
    typedef uint32_t u3 __attribute__((ext_vector_type(3)));
    typedef uint32_t u2 __attribute__((ext_vector_type(2)));
    if constexpr (WORDS == 4) {
        const u4 v = __builtin_amdgcn_raw_buffer_load_b128(r, lane_off, off, 0);
        w[0] = v[0]; w[1] = v[1]; w[2] = v[2]; w[3] = v[3];
    } else if constexpr (WORDS == 3) {
        const u3 v = __builtin_amdgcn_raw_buffer_load_b96(r, lane_off, off, 0);
        w[0] = v[0]; w[1] = v[1]; w[2] = v[2];
    } else {
        const u2 v = __builtin_amdgcn_raw_buffer_load_b64(r, lane_off, off, 0);
        w[0] = v[0]; w[1] = v[1];
    }
}

// 64 chunks of 16 bytes from memory straight into 1 KiB of LDS, lane after lane: from rsrc + lane_off + OFF to lds + OFF.
// The compiler does not know of the request: it counts in vmcnt all the same, so the compiler's own waits only get longer,
// and whoever reads the bytes waits for them (pf_arrived) before the barrier in front of the reads.
template <int OFF>
__device__ __forceinline__ void pf_load_lds(u4 rsrc, uint32_t lane_off, uint32_t lds)
{
    static_assert(OFF >= 0 && OFF < 4096 && OFF % 16 == 0, "");
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen offset:%3 lds" : : "s"(lds), "v"(lane_off), "s"(rsrc), "i"(OFF) : "memory", "m0");
}
// everything but the NEWER last requests is there
template <int NEWER>
__device__ __forceinline__ void pf_arrived()
{
    static_assert(NEWER <= 1, "");
    if constexpr (NEWER == 0) asm volatile("s_waitcnt vmcnt(0)" : : : "memory");
    else asm volatile("s_waitcnt vmcnt(1)" : : : "memory");
}
template <int V> struct PfInt { static constexpr int value = V; };
template <int N, int I = 0, typename F>
__device__ __forceinline__ void pf_for(F&& f)
{
    if constexpr (I < N) {
        f(PfInt<I>{});
        pf_for<N, I + 1>(f);
    }
}

// Stored words of one step of 64 columns, as loaded: the lane owns row (lane & 31) of the wavefront's 32 rows and the
// chunks 4q .. 4q+3 of the step, q = lane >> 5 (fp16 tiles: chunks 2i + q).
template <int FMT>
struct WReg {
    uint32_t w[Fmt<FMT>::WORDS];
};
template <>
struct WReg<S_F16> {
    u4 v[4];
};

// One segment's stored operand, seen from a lane: everything is relative to the workgroup's first row block.
struct WSeg {
    __amdgpu_buffer_rsrc_t tiles;                     // from the workgroup's first row block
    __amdgpu_buffer_rsrc_t scales;                    // from its first row
    __amdgpu_buffer_rsrc_t zeros;
    int K;
    uint32_t tile_off, scale_off, zero_off;           // the lane's byte offsets
    uint32_t gdiv, gmagic;                            // tiles of 128 columns per quantisation group, and ceil(2^32 / gdiv)
    int ng;                                           // groups per row
    bool by8;                                         // scales and zero-points eight groups at a time
};

// rb: the lane's row block, relative and clamped to a valid one
template <int FMT>
__device__ __forceinline__ void place_w(WSeg& a, int rb, int lane)
{
    const int n = lane & 15, q = lane >> 5;
    if constexpr (FMT == S_F16) a.tile_off = (uint32_t)(rb * (a.K / 32) * 64 + 16 * q + n) * 16u;
    else a.tile_off = (uint32_t)(rb * (a.K / 128) * 64 + 16 * q + n) * (4u * Fmt<FMT>::WORDS);
    a.scale_off = (uint32_t)(rb * 16 + n) * a.ng * 2u;
    a.zero_off = (uint32_t)(rb * 16 + n) * ((a.ng + 7) / 8) * 4u;
}

// step s: columns 64 s .. 64 s + 63 of the segment
template <int FMT>
__device__ __forceinline__ void load_w(WReg<FMT>& r, const WSeg& a, int s)
{
    if constexpr (FMT == S_F16) {                     // chunk 2 i + q: tile 2 s + i / 2, its columns 8 (2 (i % 2) + q) ..
#pragma unroll
        for (int i = 0; i < 4; ++i)
            r.v[i] = __builtin_amdgcn_raw_buffer_load_b128(a.tiles, a.tile_off, (uint32_t)((2 * s + (i >> 1)) * 64 + 32 * (i & 1)) * 16u, 0);
    } else {
        pf_load<Fmt<FMT>::WORDS>(r.w, a.tiles, a.tile_off, (uint32_t)((s >> 1) * 64 + 32 * (s & 1)) * (4u * Fmt<FMT>::WORDS));
    }
}

template <int FMT>
__device__ __forceinline__ void load_scale(WScale& r, const WSeg& a, int s)
{
    if constexpr (FMT != S_F16) {
        const uint32_t g = s >> 1;
        if (a.by8) {
            const u4 v = __builtin_amdgcn_raw_buffer_load_b128(a.scales, a.scale_off, (g & ~7u) * 2u, 0);
            r.s[0] = v[0]; r.s[1] = v[1]; r.s[2] = v[2]; r.s[3] = v[3];
            if constexpr (Fmt<FMT>::ASYM) r.z = __builtin_amdgcn_raw_buffer_load_b32(a.zeros, a.zero_off, (g >> 3) * 4u, 0);
        } else {
            const uint32_t grp = a.gdiv == 1 ? g : __umulhi(g, a.gmagic);
            r.s[0] = __builtin_amdgcn_raw_buffer_load_b16(a.scales, a.scale_off, grp * 2u, 0);
            if constexpr (Fmt<FMT>::ASYM) r.z = __builtin_amdgcn_raw_buffer_load_b32(a.zeros, a.zero_off, (grp >> 3) * 4u, 0);
        }
    }
}

// whether step s is the first that the values loaded before it do not cover
template <int FMT>
__device__ __forceinline__ bool scale_due(const WSeg& a, int s) { return FMT != S_F16 && (s & (a.by8 ? 15 : 1)) == 0; }

// fragment T (of four) of the lane's chunks into the slab; the group's scale is folded in (one fp16 rounding per weight).
// wl: the lane's first chunk in the slab
template <int FMT, int T>
__device__ __forceinline__ void store_w(const WReg<FMT>& r, uint32_t sraw, uint32_t z, uint32_t wl)
{
    if constexpr (FMT == S_F16) {
        *(u4*)(eora_smem + (wl ^ (T << 5))) = r.v[T];
    } else {
        const _Float16 sc = __builtin_bit_cast(_Float16, (uint16_t)sraw);
        const h8 s = {sc, sc, sc, sc, sc, sc, sc, sc};
        *(h8*)(eora_smem + (wl ^ (T << 4))) = decode_frag<T>(r.w, z) * s;
    }
}

// FM: format of the backbone (S_Q4, S_Q3, S_Q2).  FE2: S_NONE, or the format of a second segment's tiles (B): the kernel then
// continues over a second segment with its own activations (t).  TM: blocks of 32 tokens per wavefront.
template <int FM, int FE2, int TM>
__global__ __launch_bounds__(PF_NT, 2) void prefill_kernel(PrefillArgs ga)
{
    constexpr bool EXT = FE2 != S_NONE;
    constexpr int BM = pf_bm(TM), XS = BM * 128, FX = EXT ? FE2 : S_F16;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    int ntn = 0;                                                  // row tiles of all members
    for (int m = 0; m < ga.n; ++m) ntn += (ga.N[m] + PF_BN - 1) / PF_BN;
    const int ntm = (ga.M + BM - 1) / BM;
    const int tile_id = blockIdx.x % (ntn * ntm), ks = blockIdx.x / (ntn * ntm);     // ks > 0 only with ksplit > 1
    const int m0 = (tile_id / ntn) * BM;
    int nt = tile_id % ntn, mem = 0;                              // row tile within its member
    while (mem + 1 < ga.n && nt >= (ga.N[mem] + PF_BN - 1) / PF_BN) {
        nt -= (ga.N[mem] + PF_BN - 1) / PF_BN;
        ++mem;
    }
    const int M = ga.M, N = ga.N[mem], K1 = ga.K1, K2 = ga.K2;
    const int R0 = nt * (PF_BN / 16), nblk = N / 16;
    int rb = 2 * wave + ((lane >> 4) & 1);                        // the row block this lane supplies a row of, clamped to a valid one
    rb = R0 + rb < nblk ? rb : nblk - 1 - R0;
    const int H1 = K1 / 64, H2 = EXT ? K2 / 64 : 0;
    // this workgroup's steps: [sb, se) of the first segment, and with the last part the second segment's, [se, GT)
    const int sb = 2 * (ks * (H1 / 2) / ga.ksplit), se = 2 * ((ks + 1) * (H1 / 2) / ga.ksplit);
    const int GT = EXT && ks == ga.ksplit - 1 ? H1 + H2 : se;

    WSeg w1;
    w1.K = K1;
    w1.gdiv = ga.group / 128;
    w1.gmagic = w1.gdiv > 1 ? (uint32_t)((0x100000000ull + w1.gdiv - 1) / w1.gdiv) : 0u;
    w1.ng = K1 / 128 / (int)w1.gdiv;
    w1.by8 = w1.gdiv == 1 && w1.ng % 8 == 0;
    w1.tiles = pf_rsrc((const uint32_t*)ga.w[mem] + (size_t)R0 * (K1 / Fmt<FM>::KT) * 64 * Fmt<FM>::WORDS);
    w1.scales = pf_rsrc((const uint16_t*)ga.w_scales[mem] + (size_t)R0 * 16 * w1.ng);
    w1.zeros = pf_rsrc(ga.w_zeros[mem] + (size_t)R0 * 16 * ((w1.ng + 7) / 8));
    place_w<FM>(w1, rb, lane);
    WSeg w2;
    if constexpr (EXT) {
        w2.K = K2;
        w2.gdiv = 1;
        w2.gmagic = 0;
        w2.ng = K2 / 128;
        w2.by8 = false;                                           // (a rank has four groups at most)
        w2.tiles = pf_rsrc((const uint32_t*)ga.w2[mem] + (size_t)R0 * (K2 / Fmt<FX>::KT) * 64 * Fmt<FX>::WORDS);
        w2.scales = pf_rsrc((const uint16_t*)ga.w2_scales[mem] + (size_t)R0 * 16 * w2.ng);
        place_w<FX>(w2, rb, lane);
    }

    // x: a request is eight rows of 64 columns; wavefront w brings rows 8 TM w .. of the slab.  Lane l is row l / 8 of them, and the
    // chunk that belongs into slot l % 8 of that row.  Rows beyond M re-read the last one (never stored).
    constexpr int W0 = 3 * XS;                                    // LDS: three slabs of x, two of weights
    int xrow[TM];
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int row = 8 * (TM * wave + i) + (lane >> 3);
        xrow[i] = m0 + row < M ? row : M - 1 - m0;
    }
    // chunk of request i: (l % 8) ^ ((row / 2) % 8), row / 2 = 4 (TM w + i) + l / 16
    const int xc = 8 * ((lane & 7) ^ (lane >> 4));
    // the lane's byte offsets in the rows of x, shifted so that request I may name offset 1024 I on both sides
    uint32_t xo[TM];
    auto place_x = [&](int ld) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < TM; ++i) xo[i] = (uint32_t)(xrow[i] * ld + (xc ^ (((TM * wave + i) & 1) << 5))) * 2u + 1024u * (TM - 1 - i);
    };
    const uint32_t xlds = TM * wave * 1024;
    auto x_base = [&](const _Float16* p, int ld) __attribute__((always_inline)) {     // of the segment's first step
        return (uint64_t)(p + (size_t)m0 * ld) - 1024u * (TM - 1);
    };
    auto load_x = [&](auto itag, uint64_t at, uint32_t buf) __attribute__((always_inline)) {
        constexpr int I = decltype(itag)::value;
        pf_load_lds<1024 * I>(u4{(uint32_t)at, (uint32_t)(at >> 32), 0xffffffffu, 0x00027000u}, xo[I], buf + xlds);
    };

    constexpr int NX = 2 * TM;                                    // blocks of 16 tokens per wavefront; 4 blocks of 16 rows
    f4 acc[NX][4];
#pragma unroll
    for (int i = 0; i < NX; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[i][e] = f4{0.f, 0.f, 0.f, 0.f};

    // operand fragments: 16 rows x 32 columns, lane l row l % 16, columns 8 (l / 16) .. of the half step
    const uint32_t fo = pf_slot(lane & 15, lane >> 4);
    const uint32_t xf = fo + (wave & 1) * (BM / 2) * 128, wf = W0 + fo + (wave >> 1) * 64 * 128;
    h8 fx[4], fw[2][4];
#pragma unroll
    for (int i = 0; i < 4; ++i) fx[i] = h8{};
#pragma unroll
    for (int e = 0; e < 4; ++e) fw[0][e] = fw[1][e] = h8{};

    WReg<FM> wp[2];                                               // stored words of step sb + i in wp[i % 2], two steps ahead
    WScale sc;                                                    // the block's groups behind the one in use, the next one lowest
    uint32_t zsh = 0;                                             // where the next one's zero-point is
    uint32_t sraw = 0, z = 8;                                     // the group in use
    auto load_block = [&](int s) __attribute__((always_inline)) {
        load_scale<FM>(sc, w1, s);
        if (!w1.by8) zsh = 4 * ((w1.gdiv == 1 ? (uint32_t)s >> 1 : __umulhi((uint32_t)s >> 1, w1.gmagic)) & 7);
    };
    auto next_group = [&]() __attribute__((always_inline)) {
        sraw = sc.s[0];
        z = (sc.z >> zsh) & 0xFu;
        asm volatile("" : "+v"(sraw), "+v"(z));                   // (formed here: a later request replaces what they come from)
#pragma unroll
        for (int i = 0; i < 3; ++i) sc.s[i] = __builtin_amdgcn_alignbit(sc.s[i + 1], sc.s[i], 16);
        sc.s[3] >>= 16;
        sc.z >>= 4;
    };
    const int row32 = lane & 31, q = lane >> 5;
    const uint32_t wd = W0 + wave * 32 * 128 + pf_slot(row32, 4 * q);
    uint32_t xb = 0;                                              // LDS offset of the current step's slab of x
    auto turn3 = [](uint32_t b) __attribute__((always_inline)) { return b == 2 * XS ? 0u : b + XS; };

    place_x(ga.ldx);
    uint64_t xat = x_base(ga.x, ga.ldx) + (uint64_t)sb * 128;
    pf_for<TM>([&](auto i) __attribute__((always_inline)) { load_x(i, xat, 0); });
    load_w<FM>(wp[0], w1, sb);
    load_block(sb);
    pf_for<TM>([&](auto i) __attribute__((always_inline)) { load_x(i, xat + 128, XS); });
    load_w<FM>(wp[1], w1, sb + 1);
    pf_arrived<0>();
    if (w1.by8)                                                   // (a part that begins within eight groups)
        for (int e = 0; e < ((sb >> 1) & 7); ++e) next_group();
    next_group();
    pf_for<4>([&](auto t) __attribute__((always_inline)) { store_w<FM, decltype(t)::value>(wp[0], sraw, z, wd); });
    load_w<FM>(wp[0], w1, sb + 2 < se ? sb + 2 : se - 1);
    __syncthreads();
    xat += 256;                                                   // the step after next's

    // A step is 2 NX units of four MFMAs: block i of 16 tokens times the four blocks of 16 rows, for either half h of the
    // step's columns.  The fragments of four units are in registers; a unit's place is refilled right after its MFMAs.  The
    // last four units of a step are carried out behind its barrier, while the first reads of the next step are on their way.
    constexpr int U = 2 * NX;
    auto unit = [&](auto utag, auto rtag, auto wtag) __attribute__((always_inline)) {   // rtag: whether there is something to read behind it
        constexpr int u = decltype(utag)::value, h = u / NX, i = u % NX;
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[i][e] = mfma16(fw[h][e], fx[u & 3], acc[i][e]);
        if constexpr (decltype(rtag)::value) {
            constexpr int v = (u + 4) % U;                        // (behind the barrier: the next step's)
            fx[u & 3] = *(const h8*)(eora_smem + ((xf + xb) ^ ((v / NX) << 6)) + (v % NX) * 2048);
            // the other half's rows: for the second half in turn over the first, for the next step's first half behind the barrier
            constexpr int f = h == 0 && NX == 8 ? (i % 2 ? -1 : i / 2) : i - (NX - 4);
            if constexpr (f >= 0) fw[h ^ 1][f] = *(const h8*)(eora_smem + (wf ^ ((h ^ 1) << 6)) + decltype(wtag)::value * PF_WS + f * 2048);
        }
    };
    // One step (its weights are in slab PAR).  MAIN: it and the two behind it are the first segment's.  Otherwise what there is
    // to bring is found out step by step.
    WReg<FX> we;
    WScale se2;
    auto step = [&](auto main_tag, auto par_tag, int s) __attribute__((always_inline)) {
        constexpr bool MAIN = decltype(main_tag)::value != 0;
        constexpr int PAR = decltype(par_tag)::value, NXT = PAR ^ 1;
        __builtin_amdgcn_s_setprio(3);
        pf_for<4>([&](auto xtag) __attribute__((always_inline)) {
            unit(PfInt<U - 4 + decltype(xtag)::value>{}, PfInt<1>{}, PfInt<PAR>{});
            PF_SCHED();
        });
        const bool main1 = MAIN || s + 1 < se, ext1 = EXT && !MAIN && s + 1 >= se && s + 1 < GT;
        const bool main2 = MAIN || s + 2 < se, ext2 = EXT && !MAIN && s + 2 >= se && s + 2 < GT;
        // the next step's x, requested a step ago, and its stored words (those of the step behind it are the last request)
        pf_arrived<MAIN ? 1 : 0>();
#pragma unroll
        for (int i = 0; i < Fmt<FM>::WORDS; ++i) asm volatile("" : "+v"(wp[NXT].w[i]));
        if (main1 && PAR == 1) next_group();
        if (main2 && PAR == 0 && scale_due<FM>(w1, s + 2)) load_block(s + 2);
        if constexpr (EXT && !MAIN) {
            if (ext1) {                                           // (a handful of steps: all at once)
                const uint32_t wx = W0 + wave * 32 * 128 + pf_slot(row32, FX == S_F16 ? q : 4 * q) + NXT * PF_WS;
                constexpr uint32_t Z2 = FX == S_Q3S128 ? 4u : 8u;             // (symmetric formats, one group in two steps)
                store_w<FX, 0>(we, se2.s[0], Z2, wx);
                store_w<FX, 1>(we, se2.s[0], Z2, wx);
                store_w<FX, 2>(we, se2.s[0], Z2, wx);
                store_w<FX, 3>(we, se2.s[0], Z2, wx);
            }
            if (s + 2 == se && GT > se) {                         // from here on x is t
                place_x(ga.ldx2);
                xat = x_base(ga.x2[mem], ga.ldx2);
            }
            if (ext2) {
                load_w<FX>(we, w2, s + 2 - H1);
                if (scale_due<FX>(w2, s + 2 - H1)) load_scale<FX>(se2, w2, s + 2 - H1);
            }
        }
        const uint32_t xnew = turn3(turn3(xb));
        PF_SCHED();
        pf_for<U - 4>([&](auto xtag) __attribute__((always_inline)) {
            constexpr int x = decltype(xtag)::value, PER = (U - 4) / 4;
            if constexpr (x % 4 == 0) __builtin_amdgcn_s_setprio(2 - x / 4);
            unit(PfInt<x>{}, PfInt<1>{}, PfInt<PAR>{});
            // x of the step after next goes where the step before this one had its own (everyone has left it at the barrier);
            // one request at a time: a compute unit takes in 64 bytes a cycle, and a wavefront that asks for more at once waits
            if constexpr (x % PER == 0 && x / PER < TM)
                if (main2 || ext2) load_x(PfInt<x / PER>{}, xat, xnew);
            if constexpr (x % PER == PER - 1) {
                constexpr int T = x / PER;
                if (main1) store_w<FM, T>(wp[NXT], sraw, z, wd + NXT * PF_WS);
            }
            PF_SCHED();
        });
        if constexpr (MAIN) load_w<FM>(wp[NXT], w1, s + 3 < se ? s + 3 : se - 1);
        xat += 128;
        xb = turn3(xb);
        __syncthreads();
    };
    for (int s = sb; s < se - 2; s += 2) {
        step(PfInt<1>{}, PfInt<0>{}, s);
        step(PfInt<1>{}, PfInt<1>{}, s + 1);
    }
    for (int s = se - 2; s < GT; s += 2) {
        step(PfInt<0>{}, PfInt<0>{}, s);
        if (s + 1 < GT) step(PfInt<0>{}, PfInt<1>{}, s + 1);
    }
    pf_for<4>([&](auto xtag) __attribute__((always_inline)) { unit(PfInt<U - 4 + decltype(xtag)::value>{}, PfInt<0>{}, PfInt<0>{}); });

    // ---- epilogue: wavefront-private staging of 32 tokens x 64 rows, so that y is written in 128-byte rows ----------
    // result register v of lane l: row 4 (l / 16) + v of the block's 16, token l % 16
    const int tok0 = m0 + (wave & 1) * (BM / 2), o0 = R0 * 16 + (wave >> 1) * 64;
    const int tr = lane & 15, kg = lane >> 4;
    if (ga.ksplit > 1) {                                          // split contraction: this part's fp32 tile
        constexpr int TS = 68;                                    // floats per token row in the staging tile (64 + pad)
        float* const tile = (float*)eora_smem + wave * 32 * TS;
#pragma unroll
        for (int i = 0; i < TM; ++i) {
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int e = 0; e < 4; ++e) *(f4*)(tile + (16 * b + tr) * TS + 16 * e + 4 * kg) = acc[2 * i + b][e];
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int it = 0; it < 8; ++it) {
                const int tok = 4 * it + (lane >> 4), c = 4 * (lane & 15);
                const int m = tok0 + 32 * i + tok, o = o0 + c;
                const f4 v = *(const f4*)(tile + tok * TS + c);
                if (m < M && o < N) *(f4*)(ga.part + ((size_t)ks * M + m) * ga.ldp + ga.pcol[mem] + o) = v;
            }
            __builtin_amdgcn_wave_barrier();
        }
        return;
    }
    constexpr int TS = 72;                                        // halves per token row in the staging tile (64 + pad)
    typedef _Float16 h4 __attribute__((ext_vector_type(4)));
    _Float16* const tile = (_Float16*)eora_smem + wave * 32 * TS;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const f4 a = acc[2 * i + b][e];
                *(h4*)(tile + (16 * b + tr) * TS + 16 * e + 4 * kg) = h4{(_Float16)a[0], (_Float16)a[1], (_Float16)a[2], (_Float16)a[3]};
            }
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int it = 0; it < 4; ++it) {
            const int tok = 8 * it + (lane >> 3), c = 8 * (lane & 7);
            const int m = tok0 + 32 * i + tok, o = o0 + c;
            const u4 v = *(const u4*)(tile + tok * TS + c);
            if (m < M && o < N) *(u4*)((_Float16*)ga.y[mem] + (size_t)m * ga.ldy[mem] + o) = v;
        }
        __builtin_amdgcn_wave_barrier();
    }
}

template <int FM, int FE2, int TM>
static hipError_t launch_pf_tile(const PrefillArgs& a, hipStream_t stream)
{
    auto kern = prefill_kernel<FM, FE2, TM>;
    hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, pf_lds(TM));
    if (e != hipSuccess) return e;
    int ntn = 0;
    for (int m = 0; m < a.n; ++m) ntn += (a.N[m] + PF_BN - 1) / PF_BN;
    const int ntm = (a.M + pf_bm(TM) - 1) / pf_bm(TM);
    note_launch("prefill FM=%d EXT=%d ksplit=%d n=%d FE=%d", FM, (int)(FE2 != S_NONE), a.ksplit, a.n, FE2);
    note_prefill("prefill tokens=%d", pf_bm(TM));
    hipLaunchKernelGGL(kern, dim3(ntn * ntm * a.ksplit), dim3(PF_NT), pf_lds(TM), stream, a);
    return hipGetLastError();
}

template <int FM, int FE2>
static hipError_t launch_pf(const PrefillArgs& a, hipStream_t stream)
{
    switch (a.tm) {
        case 2: return launch_pf_tile<FM, FE2, 2>(a, stream);
        case 3: return launch_pf_tile<FM, FE2, 3>(a, stream);
        case 4: return launch_pf_tile<FM, FE2, 4>(a, stream);
        default: return hipErrorInvalidValue;
    }
}

// W parts behind ks, in order, their loads on their way together
template <int W>
static __device__ __forceinline__ void add_parts(const float* __restrict__ p, size_t count, int& ks, f4& v)
{
    f4 w[W];
#pragma unroll
    for (int e = 0; e < W; ++e) w[e] = *(const f4*)(p + (ks + e) * count);
#pragma unroll
    for (int e = 0; e < W; ++e) v += w[e];
    ks += W;
}

// Eight parts at a time, then what is left of them together (one by one, 32 parts of 1 MiB take 15 us, and the seven behind the first of
// eight parts cost a call of 427 tokens x 2048, rank 256 twice, 0.9 of 38.6 us; the last part again in place of those that are not
// there costs up to 2 % of a call: 318 tokens x 1280 -> 944, rank 128, ten parts, 28.8 -> 29.4 us; 333 x 14336, 38 parts, 68.4 -> 69.7)
__global__ __launch_bounds__(256) void reduce_parts_kernel(const float* __restrict__ part, _Float16* __restrict__ T, size_t count, int ksplit)
{
    const size_t i = 4 * ((size_t)blockIdx.x * 256 + threadIdx.x);
    if (i >= count) return;
    const float* __restrict__ p = part + i;
    f4 v = *(const f4*)p;
    int ks = 1;
    while (ks + 8 <= ksplit) add_parts<8>(p, count, ks, v);
    switch (ksplit - ks) {
        case 1: add_parts<1>(p, count, ks, v); break;
        case 2: add_parts<2>(p, count, ks, v); break;
        case 3: add_parts<3>(p, count, ks, v); break;
        case 4: add_parts<4>(p, count, ks, v); break;
        case 5: add_parts<5>(p, count, ks, v); break;
        case 6: add_parts<6>(p, count, ks, v); break;
        case 7: add_parts<7>(p, count, ks, v); break;
    }
    typedef _Float16 h4 __attribute__((ext_vector_type(4)));
    *(h4*)(T + i) = h4{(_Float16)v[0], (_Float16)v[1], (_Float16)v[2], (_Float16)v[3]};
}

hipError_t launch_reduce_parts(const float* part, void* T, size_t count, int ksplit, hipStream_t stream)
{
    hipLaunchKernelGGL(reduce_parts_kernel, dim3((unsigned)((count / 4 + 255) / 256)), dim3(256), 0, stream, part, (_Float16*)T, count, ksplit);
    return hipGetLastError();
}

// y of every member = fp16(sum over the parts, in order); eight columns per thread
__global__ __launch_bounds__(256) void reduce_members_kernel(PrefillArgs a)
{
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    const int per_row = a.ldp / 8;
    const int m = (int)(i / per_row), c = 8 * (int)(i - (size_t)m * per_row);
    if (m >= a.M) return;
    const size_t stride = (size_t)a.M * a.ldp;
    const float* p = a.part + (size_t)m * a.ldp + c;
    f4 v0 = *(const f4*)p, v1 = *(const f4*)(p + 4);
    for (int ks = 1; ks < a.ksplit; ++ks) {
        v0 += *(const f4*)(p + ks * stride);
        v1 += *(const f4*)(p + ks * stride + 4);
    }
    int mem = 0;
#pragma unroll
    for (int q = 1; q < MAX_GROUP; ++q)
        if (q < a.n && c >= a.pcol[q]) mem = q;
    _Float16* const y = (_Float16*)a.y[mem] + (size_t)m * a.ldy[mem] + (c - a.pcol[mem]);
    *(h8*)y = h8{(_Float16)v0[0], (_Float16)v0[1], (_Float16)v0[2], (_Float16)v0[3], (_Float16)v1[0], (_Float16)v1[1], (_Float16)v1[2], (_Float16)v1[3]};
}

hipError_t launch_reduce_members(const PrefillArgs& a, hipStream_t stream)
{
    const size_t items = (size_t)a.M * a.ldp / 8;
    hipLaunchKernelGGL(reduce_members_kernel, dim3((unsigned)((items + 255) / 256)), dim3(256), 0, stream, a);
    return hipGetLastError();
}

template <int FM>
static hipError_t launch_pf_ext(const PrefillArgs& a, int fe2, hipStream_t stream)
{
    switch (fe2) {
        case S_NONE: return launch_pf<FM, S_NONE>(a, stream);
        case S_F16: return launch_pf<FM, S_F16>(a, stream);
        case S_Q4S128: return launch_pf<FM, S_Q4S128>(a, stream);
        case S_Q3S128: return launch_pf<FM, S_Q3S128>(a, stream);
        default: return hipErrorInvalidValue;
    }
}

// fe2: S_NONE, or the format of the second segment's tiles
hipError_t launch_prefill(const PrefillArgs& a, int fm, int fe2, hipStream_t stream)
{
    if (a.by128) return launch_prefill128(a, fm, fe2, stream);
    switch (fm) {
        case S_Q4: return launch_pf_ext<S_Q4>(a, fe2, stream);
        case S_Q3: return launch_pf_ext<S_Q3>(a, fe2, stream);
        case S_Q2: return launch_pf_ext<S_Q2>(a, fe2, stream);
        default: return hipErrorInvalidValue;
    }
}

// T[m][c] = 0 wherever column c does not belong to the adapter of token row m (several adapters side by side)
__global__ __launch_bounds__(256) void mask_t_kernel(_Float16* __restrict__ T, const int* __restrict__ adapter, int M, int R, int r_per)
{
    const size_t i = 8 * ((size_t)blockIdx.x * 256 + threadIdx.x);       // eight columns of one row (R and r_per are multiples of 8)
    if (i >= (size_t)M * R) return;
    const int m = (int)(i / R), c = (int)(i % R);
    if (adapter[m] != c / r_per) *(u4*)(T + i) = u4{0u, 0u, 0u, 0u};
}

hipError_t launch_mask_t(void* T, const int* adapter, int M, int R, int r_per, hipStream_t stream)
{
    const size_t chunks = (size_t)M * R / 8;
    hipLaunchKernelGGL(mask_t_kernel, dim3((unsigned)((chunks + 255) / 256)), dim3(256), 0, stream, (_Float16*)T, adapter, M, R, r_per);
    return hipGetLastError();
}

}  // namespace eora
