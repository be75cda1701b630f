// C-ABI entry points: argument validation and the static choice of kernel.  No device memory is
// allocated here and nothing is kept between calls.
#include "eora.h"
#include "kernels.hpp"

#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <mutex>

namespace eora {

namespace {
struct LaunchNote { const char* fmt; int v[8]; };
LaunchNote g_last_launch = {nullptr, {0, 0, 0, 0, 0, 0, 0, 0}};
}  // namespace

void note_launch(const char* fmt, int a, int b, int c, int d, int e, int f, int g, int h) { g_last_launch = {fmt, {a, b, c, d, e, f, g, h}}; }

namespace {
LaunchNote g_last_prefill = {nullptr, {0, 0, 0, 0, 0, 0, 0, 0}};
}  // namespace

void note_prefill(const char* fmt, int tokens) { g_last_prefill = {fmt, {tokens, 0, 0, 0, 0, 0, 0, 0}}; }

}  // namespace eora

namespace {

using namespace eora;

constexpr size_t WS_HEADER = 270336;       // counters and flags (HDR_WORDS 32-bit words)
constexpr int MAX_RANK = 512;
constexpr int CHUNK_TOKENS = 16 * MAX_YBLOCKS;      // tokens per launch of the small-M kernels
constexpr int PREFILL_MIN_TOKENS = 128;             // from here on the GEMM kernel takes over
static_assert(HDR_WORDS * 4 <= WS_HEADER, "header too small");

int g_spin_limit = 1 << 22;                // bounded wait of the up-projection (about a second)

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
inline size_t round256(size_t v) { return (v + 255) & ~(size_t)255; }

int check_backbone_shape(int M, int d_in, int d_out, int r)
{
    if (M < 0 || d_in <= 0 || d_out <= 0 || r < 0) return EORA_ERR_SHAPE;
    if (d_out % 16 || d_in % 128 || r > MAX_RANK) return EORA_ERR_SHAPE;
    return EORA_OK;
}

// Set EORA_VERBOSE=1 to have a refused launch explain itself on stderr.
bool failed(hipError_t e, const char* what)
{
    if (e == hipSuccess) return false;
    static const bool verbose = getenv("EORA_VERBOSE") != nullptr;      // read once per process
    if (verbose) fprintf(stderr, "eora: %s: %s\n", what, hipGetErrorString(e));
    return true;
}

int check_group(int d_in, int group)
{
    if (group <= 0 || group % 128 || d_in % group) return EORA_ERR_SHAPE;
    return EORA_OK;
}

// workspace = header | tagged partials of t | fp32 partials (sparse.hip) | t (fp16, prefill) or partial outputs.
// The regions sit at fixed offsets whatever (M, r) a call has, so that calls of different shapes on one
// workspace never read one region's bytes as another's.  (token blocks) x kcn <= 32 and r <= 512.
constexpr size_t MAX_PART_ELEMS = 32 * 16 * 512;
constexpr size_t WS_PAIRS = WS_HEADER;
constexpr size_t WS_PARTS = WS_PAIRS + MAX_PART_ELEMS * 8;
constexpr size_t WS_T = WS_PARTS + MAX_PART_ELEMS * 4;
// fp32 partial outputs of a quantised call of 5 .. 127 tokens whose contraction is cut into parts in different workgroups
constexpr size_t WIDE_SPLIT_BYTES = 12u << 20;

// one launch of the kernel for 5 .. 16 tokens (x resident in LDS) for validated members that share x; the caller has
// checked stream_fits
int launch_stream_group(const void* x, const eora_q_member* members, int n, int M, int d_in, int r, int w_bits,
                        int fa, int fe, void* workspace, hipStream_t stream, const int* adapter = nullptr, int r_per = 0)
{
    StreamArgs a{};
    a.x = (const _Float16*)x;
    for (int m = 0; m < 4; ++m) {
        const eora_q_member& e = members[m < n ? m : 0];
        a.w[m] = e.qweight;
        a.w_scales[m] = (const _Float16*)e.scales;
        a.w_zeros[m] = (const uint32_t*)e.qzeros;
        a.A[m] = e.A;
        a.A_scales[m] = (const _Float16*)e.A_scales;
        a.B[m] = e.B;
        a.B_scales[m] = (const _Float16*)e.B_scales;
        a.y[m] = (_Float16*)e.y;
        a.d_out[m] = m < n ? e.d_out : 0;
    }
    a.n = n;
    a.hdr = (uint32_t*)workspace;
    a.tpair = (unsigned long long*)((char*)workspace + WS_PAIRS);
    a.M = M;
    a.d_in = d_in;
    a.r = r;
    a.spin_limit = g_spin_limit;
    a.adapter = adapter;
    a.r_per = r_per;
    if (failed(launch_stream(a, backbone_format(w_bits), fa, fe, stream), "linear_q (stream)")) return EORA_ERR_LAUNCH;
    return EORA_OK;
}

// the kernel for 5 and more tokens for validated members that share x, in launches of at most CHUNK_TOKENS tokens
int launch_wide_group(const void* x, const eora_q_member* members, int n, int M, int d_in, int r, int w_bits, int group,
                      int fa, int fe, void* workspace, size_t workspace_bytes, hipStream_t stream, const int* adapter = nullptr, int r_per = 0)
{
    for (int m0 = 0; m0 < M; m0 += CHUNK_TOKENS) {
        WideArgs a{};
        a.x = (const _Float16*)x + (size_t)m0 * d_in;
        for (int m = 0; m < n; ++m) {
            const eora_q_member& e = members[m];
            a.w[m] = e.qweight;
            a.w_scales[m] = (const _Float16*)e.scales;
            a.w_zeros[m] = (const uint32_t*)e.qzeros;
            a.A[m] = e.A;
            a.A_scales[m] = (const _Float16*)e.A_scales;
            a.B[m] = e.B;
            a.B_scales[m] = (const _Float16*)e.B_scales;
            a.y[m] = (_Float16*)e.y + (size_t)m0 * e.d_out;
            a.d_out[m] = e.d_out;
        }
        a.n = n;
        a.fa = fa;
        a.fe = fe;
        a.hdr = (uint32_t*)workspace;
        a.tpair = (unsigned long long*)((char*)workspace + WS_PAIRS);
        a.tpair_count = MAX_PART_ELEMS;
        a.ypart = (float*)((char*)workspace + WS_T);
        a.ypart_count = M < PREFILL_MIN_TOKENS && workspace_bytes >= WS_T + WIDE_SPLIT_BYTES ? WIDE_SPLIT_BYTES / sizeof(float) : 0;
        a.M = M - m0 < CHUNK_TOKENS ? M - m0 : CHUNK_TOKENS;
        a.d_in = d_in;
        a.r = r;
        a.group = group;
        a.spin_limit = g_spin_limit;
        a.adapter = adapter ? adapter + m0 : nullptr;
        a.r_per = r_per;
        if (M <= 4 && !wide_q_shares_launch(a)) {         // (a longer call's last launch may have as few tokens: it promises no bits)
            for (int m = 0; m < n; ++m) {
                const int rc = launch_wide_group(x, &members[m], 1, M, d_in, r, w_bits, group, fa, fe, workspace, workspace_bytes, stream, adapter, r_per);
                if (rc != EORA_OK) return rc;
            }
            return EORA_OK;
        }
        if (failed(launch_wide_q(a, backbone_format(w_bits), stream), "linear_q (wide)")) return EORA_ERR_LAUNCH;
    }
    return EORA_OK;
}

// factor formats of the (r, ab_bits) a call names
int factor_formats(int r, int ab_bits, int* fa, int* fe)
{
    *fa = *fe = S_NONE;
    if (r == 0) return EORA_OK;
    if (ab_bits == 16) {
        if (r % 32) return EORA_ERR_SHAPE;
        *fa = *fe = S_F16;
    } else if (ab_bits == 4) {
        if (r != 64 && r % 128) return EORA_ERR_SHAPE;
        *fe = (r == 64) ? S_Q4S64 : S_Q4S128;
        *fa = S_Q4S128;
    } else if (ab_bits == 3) {
        if (r % 128) return EORA_ERR_SHAPE;
        *fa = *fe = S_Q3S128;
    } else {
        return EORA_ERR_UNSUPPORTED;
    }
    return EORA_OK;
}

// k-ranges of the down-projection: many for few tokens (every consumer adds the partials itself),
// a divisor of the number of 128-wide k-tiles
int pick_kcn(int M, int d_in)
{
    // (token blocks) x kcn <= 32: the partials' region is sized for that
    const int yblocks = ((M < CHUNK_TOKENS ? M : CHUNK_TOKENS) + 15) / 16;
    int cap = 32 / yblocks < MAX_KCN ? 32 / yblocks : MAX_KCN;
    // with more than 4 tokens every consumer reads (tokens x r x kcn) partials: few ranges
    // (a long contraction at many tokens keeps eight: its producers would otherwise take longer than the launch
    // streams; measured on the 28672- and 14336-long down projections at 64 tokens, 73.4 -> 69.3 and 40.5 -> 39.1 us)
    if (M > 4 && cap > 4 && !(M > 16 && d_in > 8192)) cap = 4;
    int kcn = 1;
    for (int c = 2; c <= cap; ++c)
        if ((d_in / 128) % c == 0) kcn = c;
    return kcn;
}

// Parts the prefill down-projection t = x.A^T (few output tiles: r / 128 per 128 tokens) splits its
// contraction into so that the launch fills the chip; their fp32 tiles are added in a fixed order.
int pick_ksplit(int M, int d_in, int r)
{
    if (r == 0) return 1;
    const int tiles = ((M + 127) / 128) * ((r + 255) / 256), G = d_in / 128;       // the GEMM kernel's tile is 128 x 256
    int want = (256 + tiles - 1) / tiles;
    want = want > 8 ? 8 : want;
    int ks = 1;
    for (int c = 2; c <= want; ++c)
        if (G % c == 0) ks = c;
    return ks;
}

// Many tokens: MFMA-bound GEMM (t = x.A^T first, then one GEMM over d_in and r)
// (fp16, 4-bit or 3-bit factors; the rank in whole steps of 128)
bool prefill_fits(int M, int r, int ab_bits) { return M >= PREFILL_MIN_TOKENS && (r == 0 || r % 128 == 0) && (ab_bits == 16 || ab_bits == 4 || ab_bits == 3 || r == 0); }

// scratch of the prefill path for n members: t (fp16, M x n*r) and the fp32 parts of its split contraction
size_t prefill_scratch_bytes(int M, int d_in, int r, int n)
{
    const int ks = pick_ksplit(M, d_in, n * r);
    return round256((size_t)M * n * r * 2) + (ks > 1 ? (size_t)ks * M * n * r * sizeof(float) : 0);
}

// the most that prefill_scratch_bytes() names for up to M tokens and ranks (n members: r = their sum) up to r: fewer tokens
// or columns of t may be cut into more parts (a workspace of the size of the largest call serves smaller ones too)
size_t prefill_scratch_most(int M, int d_in, int r)
{
    size_t parts = 0;
    for (int m = 128, last = 0; !last && m <= 256 * 128; m += 128) {          // (beyond 256 tiles nothing is cut)
        last = m >= M;
        const int tokens = last ? M : m;
        for (int q = 128; q < r + 128; q += 128) {
            const int cols = q < r ? q : r, ks = pick_ksplit(tokens, d_in, cols);
            const size_t need = ks > 1 ? (size_t)ks * tokens * cols * sizeof(float) : 0;
            parts = need > parts ? need : parts;
        }
    }
    return round256((size_t)M * r * 2) + parts;
}

// room for the fp32 partial outputs of a prompt whose contraction is cut into parts
constexpr size_t PREFILL_SPLIT_BYTES = 48u << 20;

// Parts of the launch for t that are taken: pick_ksplit's eight and a divisor of the groups leave long contractions with few
// tokens long chains of steps (333 tokens, rank 128, d_in 14336: 24 workgroups of 28 steps, 28 us).  The cheapest by rounds
// of 256 workgroups, 0.9 us a step of 64 columns and 5 a workgroup, the parts written and read at 2 TB/s and 4 us for their
// sum, as far as the workspace has room for the parts (it always has it for pick_ksplit's).  The parts cost more than the two
// kernels show, because the caches are written back between them: 2048 tokens, rank 256, d_in 14336 in 8 parts 262 us a call
// with the main GEMM, in 14 (which 4 TB/s would take) 267, and the kernels' own times say the opposite.  Contractions of up to
// 24 groups take pick_ksplit's parts at least, if these are one round: their parts are small and stay in the caches, and 2 TB/s
// would leave them whole or in too few (1262 tokens, rank 256 twice, d_in 1280: 45.2 us a call in two parts, 40.3 in five; 1194, rank
// 128 three times, d_in 1024: 39.0 whole, 36.0 in eight; 2028, rank 128 twice, d_in 2688: 52.7 in three, 51.0 in seven; 1207, rank
// 256 twice, d_in 2304: 56.7 in three, 54.4 in six; 29 shapes of 13 .. 24 groups 0.986 on average, 1.007 at most).  With 32 groups
// single calls lose 2 %.  In two rounds it is no gain (1384, rank 256 three times, d_in 1024, eight
// parts of 33 workgroups: 52.1 us, whole 45.7).
int pick_t_parts(int M, int d_in, int r, int n, size_t room)
{
    const int G = d_in / 128, tiles = ((M + 127) / 128) * n * ((r + 255) / 256), least = pick_ksplit(M, d_in, n * r);
    int best = least;
    float best_us = 1e30f;
    for (int ks = G <= 24 && tiles * least <= 256 ? least : 1; ks <= G && ks <= 64; ++ks) {
        const size_t bytes = ks > 1 ? (size_t)ks * M * n * r * sizeof(float) : 0;
        if (ks > least && bytes > room) break;
        const int steps = 2 * ((G + ks - 1) / ks);
        const float us = (float)((tiles * ks + 255) / 256) * (0.9f * steps + 5.f) + (ks > 1 ? 4.f + (float)bytes * 2.f / 2e6f : 0.f);
        if (us < best_us) {
            best_us = us;
            best = ks;
        }
    }
    return best;
}

// Tokens per workgroup (64 tm) and parts of the main GEMM's contraction.  A workgroup is 64 tm tokens x 256 rows, one per
// compute unit.  More tokens share the decoding of a weight, but a launch of few output tiles leaves most of the chip idle for
// the length of a contraction (333 tokens of the 8B layer: 32 tiles for a 4096 x 4096 linear), and tokens that are not there
// cost as much as others.  The cheapest by rounds of 256 workgroups: STEP_US a step of 64 columns and TILE_US a tile for tm = 2, 3,
// 4; the parts' fp32 outputs written and read at 11 TB/s (they stay in the caches), and 10 us for the launch that sums them, with
// the caches written back in between; 7 where a part's outputs are 2 MiB or less (192 tokens x 1024 -> 816, rank 256: 32.0 us
// whole, 30.8 in two parts).  The line is drawn for one part, not for all of them: else a part would be saved to stay below it (378 x
// 1280 -> 1008, rank 128: 31.3 us in three parts, 32.3 in two).
// The constants are fitted to calls of 402 shapes (128 .. 8192 tokens, d_in 1024 .. 28672, every tm and one to eight parts of each
// timed) for the choice they lead to, not for the times; over 722, part of them the same, it takes 1.005 times as long as the best one
// on average, 1.14 at most; with the constants of the next lines 1.011 and 1.29.
// With 5 us for the sums, 8 for a tile and 1.05, 1.25, 1.5 a step short contractions were cut that are faster whole: d_in
// 1024, 1408 tokens x 656 rows bare 16.5 -> 19.1 us in two parts; 1152, 276 x 6880, rank 128 34.2 -> 38.1 in three.  Long ones
// gain as before: 333 tokens x 14336 -> 4096 bare 153 us whole, 54 in eight parts.
// Without factors a step with 128 tokens is reckoned at BARE_STEP_US: tiles of 128 tokens in fewer parts win there where the same step
// as with factors took more parts of larger tiles (512 x 4096 -> 4096 + 1024 + 1024: 41.5 us in four parts of 256 tokens, 40.5 in
// two; 968 x 3072 -> 688 + 1040 + 1424 35.7 and 33.9; 595 x 2048 -> 5952 30.2 in two parts and 28.7 whole).
// room: bytes for the partial outputs; the parts never need more.  d_out: the members' rows.
struct PrefillTiles {
    int tm, parts;
};

// prefill.hip addresses the rows of x in a tile with 32-bit byte offsets from its first one (prefill128.hip with 64 bits): some
// eight million columns with 256 tokens
bool near_rows(int tm, int d_in) { return ((size_t)(64 * tm - 1) * d_in + 64) * 2 + 4096 <= 0xFFFFFFFFull; }

PrefillTiles pick_prefill(int M, int d_in, int r, const int* d_out, int n, size_t room)
{
    static const float STEP_US[5] = {0.f, 0.f, 0.97f, 1.18f, 1.21f}, TILE_US[5] = {0.f, 0.f, 3.f, 4.f, 8.f};
    constexpr float BARE_STEP_US = 0.9f;
    const int G = d_in / 128;
    size_t rows = 0;
    int row_tiles = 0;
    for (int m = 0; m < n; ++m) {
        rows += d_out[m];
        row_tiles += (d_out[m] + 255) / 256;
    }
    PrefillTiles best{2, 1};
    float best_us = 1e30f;
    for (int ks = 1; ks <= 8 && (ks == 1 || ks * 4 <= G + 3); ++ks) {
        const size_t bytes = (size_t)ks * M * rows * sizeof(float);
        if (ks > 1 && bytes > room) break;                // (whole numbers: a float would round the room up to the need)
        for (int tm = 2; tm <= 4 && (tm == 2 || near_rows(tm, d_in)); ++tm) {
            const size_t wgs = (size_t)row_tiles * ((M + 64 * tm - 1) / (64 * tm)) * ks;
            const float step_us = tm == 2 && r == 0 ? BARE_STEP_US : STEP_US[tm];
            const float us = (float)((wgs + 255) / 256) * (step_us * (2 * ((G + ks - 1) / ks) + r / 64) + TILE_US[tm]) +
                             (ks > 1 ? ((size_t)M * rows * sizeof(float) <= 2u << 20 ? 7.f : 10.f) + (float)bytes * 2.f / 11e6f : 0.f);
            if (us < best_us) {
                best_us = us;
                best = {tm, ks};
            }
        }
    }
    return best;
}

// What the launches of a prompt do with a workspace of so many bytes (n linears of d_out[..] rows that share x)
struct PrefillPlan {
    int tm, parts, t_parts;
    bool by128;               // tm == 2: the kernel of prefill128.hip
    size_t own, main_at;      // where the fp32 parts of t and of the main GEMM begin
};
PrefillPlan plan_prefill(int M, int d_in, int r, const int* d_out, int n, size_t workspace_bytes)
{
    PrefillPlan p;
    // room for partial outputs: what is left behind t, as far as every workspace of the right size has it (the order of the
    // sums, and with it the bits of t and y, is then the same whatever larger size it has).  t's parts are there first, and
    // after their sum those of the main GEMM (2048 tokens, rank 256, 14336 -> 4096: two parts of 128 workgroups with 256 tokens
    // need the bytes of both, 265 -> 238 us).  A workspace that ends with t's own least parts has no room for the others: the
    // contraction stays whole, as for every call with a workspace of the least size
    const size_t t_bytes = round256((size_t)M * n * r * 2);
    p.own = WS_T + t_bytes;
    const size_t least = prefill_scratch_bytes(M, d_in, r, n) - t_bytes, most = least + PREFILL_SPLIT_BYTES;
    const size_t left = workspace_bytes > p.own ? workspace_bytes - p.own : 0, room = left < most ? left : most;
    p.t_parts = r > 0 ? pick_t_parts(M, d_in, r, n, room) : 1;
    const PrefillTiles t = pick_prefill(M, d_in, r, d_out, n, left > round256(least) ? room : 0);
    p.tm = t.tm;
    p.parts = t.parts;
    // The main GEMM's parts go behind t's where the workspace has the bytes of both, else in their place: written over lines that the
    // other XCDs' caches have just read, they take longer (427 tokens x 2048 -> 752 + 512, rank 256: 37.7 us a call in t's place, 34.8 behind)
    size_t rows = 0;
    for (int m = 0; m < n; ++m) rows += d_out[m];
    const size_t t_parts_bytes = p.t_parts > 1 ? round256((size_t)p.t_parts * M * n * r * sizeof(float)) : 0;
    const size_t main_bytes = p.parts > 1 ? (size_t)p.parts * M * rows * sizeof(float) : 0;
    p.main_at = p.own + (t_parts_bytes + main_bytes <= left ? t_parts_bytes : 0);
    // 128 tokens: on a partly filled chip the shorter steps of prefill128.hip win, with (nearly) all compute units busy the card's
    // power decides, and the 16x16x32 MFMAs of prefill.hip win.  Time of a call with factors on prefill.hip over that on prefill128.hip,
    // 722 shapes: up to 128 workgroups 1.037, 129 .. 192 1.019, 193 .. 224 1.003, 225 .. 248 0.994, 249 .. 256 0.983, 257 .. 384 0.997, 385 .. 448
    // 0.985, 449 .. 512 0.977, more 1.008.  Where 128 tokens are the cheapest tile, lines by how full the rounds are gain 0.1 %.
    // (pick_prefill reckons with one length of a step for both.)  Without factors prefill128.hip wins with all compute units busy too
    // once a tile has 32 steps: beyond the line 1.06 on average (1024 tokens x 28672 -> 8192, w3: 453 and 432 us; 793 x 3072 ->
    // 8784 + 5056 + 3840, w2: 106.3 and 94.1), 1.00 with fewer steps.
    size_t wgs = 0;
    for (int m = 0; m < n; ++m) wgs += (d_out[m] + 255) / 256;
    wgs *= (size_t)((M + 127) / 128) * p.parts;
    const bool long_bare = r == 0 && 2 * ((d_in / 128 + p.parts - 1) / p.parts) >= 32;
    p.by128 = p.tm == 2 && (wgs <= 248 || long_bare || !near_rows(2, d_in));
    return p;
}

// validated members that share x, as GEMMs: one launch for every member's t (the members' A side by side), one
// for every member's y
int launch_prefill_group(const void* x, const eora_q_member* members, int n, int M, int d_in, int r, int w_bits, int group,
                         int fa, int fe, const int* adapter, int r_per, void* workspace, size_t workspace_bytes, hipStream_t stream)
{
    _Float16* T = (_Float16*)((char*)workspace + WS_T);           // M x (n * r): member m owns columns m*r ..
    int d_outs[MAX_GROUP] = {0, 0, 0, 0};
    for (int m = 0; m < n; ++m) d_outs[m] = members[m].d_out;
    const PrefillPlan plan = plan_prefill(M, d_in, r, d_outs, n, workspace_bytes);
    if (r > 0) {
        PrefillArgs p{};
        p.x = (const _Float16*)x; p.ldx = d_in;
        p.group = 128;
        p.M = M; p.K1 = d_in;
        p.n = n;
        p.ksplit = plan.t_parts;
        p.part = (float*)((char*)workspace + plan.own);
        p.ldp = n * r;
        p.tm = 2;
        p.by128 = true;                                           // (few output tiles)
        for (int m = 0; m < n; ++m) {
            p.w[m] = members[m].A;
            p.w_scales[m] = (const _Float16*)members[m].A_scales;
            p.y[m] = T + (size_t)m * r; p.ldy[m] = n * r;
            p.N[m] = r; p.pcol[m] = m * r;
        }
        if (failed(launch_prefill(p, fa, S_NONE, stream), "prefill down-projection")) return EORA_ERR_LAUNCH;
        if (p.ksplit > 1 && failed(launch_reduce_parts(p.part, T, (size_t)M * n * r, p.ksplit, stream), "prefill down-projection sum"))
            return EORA_ERR_LAUNCH;
        // several adapters side by side (one member): a token row keeps its own adapter's columns of t
        if (adapter && failed(launch_mask_t(T, adapter, M, n * r, r_per, stream), "prefill adapter mask")) return EORA_ERR_LAUNCH;
    }
    PrefillArgs p{};
    p.x = (const _Float16*)x; p.ldx = d_in;
    p.group = group;
    p.M = M; p.K1 = d_in; p.K2 = r;
    p.ldx2 = n * r;
    p.n = n;
    p.ksplit = plan.parts;
    p.tm = plan.tm;
    p.by128 = plan.by128;
    p.part = (float*)((char*)workspace + plan.main_at);
    for (int m = 0; m < n; ++m) {
        p.pcol[m] = p.ldp;
        p.ldp += members[m].d_out;
        p.w[m] = members[m].qweight;
        p.w_scales[m] = (const _Float16*)members[m].scales;
        p.w_zeros[m] = (const uint32_t*)members[m].qzeros;
        p.x2[m] = T + (size_t)m * r;
        p.w2[m] = members[m].B;
        p.w2_scales[m] = (const _Float16*)members[m].B_scales;
        p.y[m] = members[m].y; p.ldy[m] = members[m].d_out;
        p.N[m] = members[m].d_out;
    }
    if (failed(launch_prefill(p, backbone_format(w_bits), r > 0 ? fe : S_NONE, stream), "prefill")) return EORA_ERR_LAUNCH;
    if (p.ksplit > 1 && failed(launch_reduce_members(p, stream), "prefill sum")) return EORA_ERR_LAUNCH;
    return EORA_OK;
}

// one launch of the decode kernel for validated members that share x
int launch_group(const void* x, const eora_q_member* members, int n, int M, int d_in, int r, int w_bits, int group,
                 int fa, int fe, int nw, int nq, void* workspace, hipStream_t stream, const int* adapter = nullptr, int r_per = 0)
{
    if (M == 0) return EORA_OK;
    GroupArgs a{};
    a.x = (const _Float16*)x;
    for (int m = 0; m < n; ++m) {
        a.w[m] = members[m].qweight;
        a.w_scales[m] = (const _Float16*)members[m].scales;
        a.w_zeros[m] = (const uint32_t*)members[m].qzeros;
        a.A[m] = members[m].A;
        a.A_scales[m] = (const _Float16*)members[m].A_scales;
        a.B[m] = members[m].B;
        a.B_scales[m] = (const _Float16*)members[m].B_scales;
        a.y[m] = (_Float16*)members[m].y;
        a.d_out[m] = members[m].d_out;
    }
    a.n = n;
    a.hdr = (uint32_t*)workspace;
    a.tpair = (unsigned long long*)((char*)workspace + WS_PAIRS);
    a.M = M;
    a.d_in = d_in;
    a.r = r;
    a.group = group;
    a.kcn = pick_kcn(M, d_in);
    if (r > 128) {
        // Large ranks: fewer k-ranges.  Every consumer reads r x kcn pairs of t and there are (r / 16) x kcn producers:
        // at most 1024 pairs per consumer, but no range longer than 4096 columns (measured on the 8B layer with 4-bit
        // factors, 7 launches: rank 512 90.9 -> 73.1 us, rank 256 67.1 -> 61.5 us; rank 128 is faster with eight).
        int cap = 1024 / r < 2 ? 2 : 1024 / r;
        while (cap * 4096 < d_in) cap *= 2;
        while (a.kcn > cap && a.kcn % 2 == 0) a.kcn /= 2;
    }
    a.spin_limit = g_spin_limit;
    a.adapter = adapter;
    a.r_per = r_per;
    a.c2n = -1;
    if (failed(launch_small(a, backbone_format(w_bits), fa, fe, nw, nq, stream), "linear_q (decode)")) return EORA_ERR_LAUNCH;
    return EORA_OK;
}

// the least a call works with: a quantised call of 5 .. 127 tokens with less than eora_workspace_bytes() never cuts its
// contraction
size_t workspace_min_bytes(int M, int d_in, int d_out, int r)
{
    return WS_T + (M >= PREFILL_MIN_TOKENS ? prefill_scratch_bytes(M, d_in, r, 1) : sparse_split_bytes(M, d_in, d_out));
}

size_t workspace_group_min_bytes(int M, int d_in, int r, int n)
{
    return WS_T + (M >= PREFILL_MIN_TOKENS ? prefill_scratch_bytes(M, d_in, r, n) : 0);
}

// what a quantised call (r: the ranks of its members together) makes use of: t of the prefill GEMM and its parts, and the
// room for partial outputs.  Never shrinks as M or r grows.
size_t workspace_room(int M, int d_in, int r)
{
    if (M >= PREFILL_MIN_TOKENS) return WS_T + prefill_scratch_most(M, d_in, r) + PREFILL_SPLIT_BYTES;
    return WS_T + (M > 4 ? WIDE_SPLIT_BYTES : 0);
}

}  // namespace

extern "C" {

size_t eora_workspace_bytes(int M, int d_in, int d_out, int r)
{
    if (check_backbone_shape(M, d_in, d_out, r) != EORA_OK) return 0;
    // partials of t for the small-M kernels (and, for a 2:4 call with a long contraction at 5 .. 127 tokens, the partial
    // outputs of its ranges); for more tokens what any smaller number asks for, too
    const int few = M < PREFILL_MIN_TOKENS ? M : PREFILL_MIN_TOKENS - 1;
    const size_t base = workspace_min_bytes(few, d_in, d_out, r), all = workspace_room(M, d_in, r);
    return base > all ? base : all;
}

size_t eora_workspace_bytes_group(int M, int d_in, int r, int n_members)
{
    if (n_members < 1 || n_members > MAX_GROUP || check_backbone_shape(M, d_in, 16, r) != EORA_OK) return 0;
    return workspace_room(M, d_in, n_members * r);
}

int eora_workspace_init(void* workspace, size_t workspace_bytes, void* stream)
{
    if (!workspace) return EORA_ERR_NULL;
    if (!aligned16(workspace)) return EORA_ERR_ALIGN;
    if (workspace_bytes < WS_HEADER) return EORA_ERR_WORKSPACE;
    // everything is cleared, not only the header: the tagged partials must not hold a leftover word
    // that reads as the tag of a coming launch
    if (workspace_bytes / 4 > 0x7fffffffull) return EORA_ERR_WORKSPACE;
    // The epoch does not start at 0: tags and flags are compared with epoch + 1, and memory that held a workspace
    // before (freed and handed out again) may still sit in a cache with that incarnation's tags.  Every
    // initialisation in this process starts from its own range of 2^20 epochs, so a tag never means two things.
    static std::atomic<uint32_t> incarnation{0};
    const uint32_t epoch0 = ((incarnation.fetch_add(1) + 1u) & 0xFFFu) << 20;
    if (failed(launch_clear_words((uint32_t*)workspace, (int)(workspace_bytes / 4), epoch0, (hipStream_t)stream), "workspace_init"))
        return EORA_ERR_LAUNCH;
    return EORA_OK;
}

int eora_workspace_error(const void* workspace, void* stream)
{
    if (!workspace) return EORA_ERR_NULL;
    uint32_t flag = 0;
    if (hipMemcpyAsync(&flag, (const uint32_t*)workspace + HDR_ERROR, sizeof(flag), hipMemcpyDeviceToHost,
                       (hipStream_t)stream) != hipSuccess)
        return EORA_ERR_LAUNCH;
    if (hipStreamSynchronize((hipStream_t)stream) != hipSuccess) return EORA_ERR_LAUNCH;
    return flag ? EORA_ERR_TIMEOUT : EORA_OK;
}

void eora_debug_set_spin_limit(int iterations) { g_spin_limit = iterations < 0 ? -1 : iterations; }

void eora_debug_set_resident_min_blocks(int blocks) { set_resident_min_blocks(blocks); }

int eora_debug_probe(int kind, const void* src, size_t bytes, void* sink, void* stream)
{
    if (!sink) return EORA_ERR_NULL;
    if (!aligned16(sink)) return EORA_ERR_ALIGN;
    if (kind == 0) {
        if (failed(launch_probe_empty((uint32_t*)sink, (hipStream_t)stream), "probe (empty)")) return EORA_ERR_LAUNCH;
        return EORA_OK;
    }
    if (kind != 1) return EORA_ERR_UNSUPPORTED;
    if (!src) return EORA_ERR_NULL;
    if (!aligned16(src)) return EORA_ERR_ALIGN;
    if (bytes == 0 || bytes % 32768 || bytes / 32768 > 0x7fffffffull) return EORA_ERR_SHAPE;
    if (failed(launch_probe_stream(src, bytes, (uint32_t*)sink, (hipStream_t)stream), "probe (stream)")) return EORA_ERR_LAUNCH;
    return EORA_OK;
}

int eora_debug_prefill_parts(int M, int d_in, int d_out, int r, size_t room)
{
    const int rc = check_backbone_shape(M, d_in, d_out, r);
    if (rc != EORA_OK) return rc;
    return pick_prefill(M, d_in, r, &d_out, 1, room).parts;
}

int eora_debug_prefill_plan(int M, int d_in, const int* d_out, int n_members, int r, size_t workspace_bytes, int* plan)
{
    if (!d_out || !plan) return EORA_ERR_NULL;
    if (n_members < 1 || n_members > MAX_GROUP) return EORA_ERR_SHAPE;
    for (int m = 0; m < n_members; ++m) {
        const int rc = check_backbone_shape(M, d_in, d_out[m], r);
        if (rc != EORA_OK) return rc;
    }
    if (M < PREFILL_MIN_TOKENS || r % 128) return EORA_ERR_SHAPE;
    const PrefillPlan p = plan_prefill(M, d_in, r, d_out, n_members, workspace_bytes);
    plan[0] = 64 * p.tm;
    plan[1] = p.parts;
    plan[2] = p.t_parts;
    plan[3] = p.by128;
    plan[4] = p.main_at == p.own && p.parts > 1 && p.t_parts > 1;
    return EORA_OK;
}

static int write_note(const LaunchNote& n, char* out, size_t capacity)
{
    if (!out || capacity == 0) return EORA_ERR_NULL;
    if (!n.fmt) {
        out[0] = 0;
        return EORA_OK;
    }
    snprintf(out, capacity, n.fmt, n.v[0], n.v[1], n.v[2], n.v[3], n.v[4], n.v[5], n.v[6], n.v[7]);
    return EORA_OK;
}

int eora_debug_last_launch(char* out, size_t capacity) { return write_note(g_last_launch, out, capacity); }

int eora_debug_last_prefill(char* out, size_t capacity) { return write_note(g_last_prefill, out, capacity); }

// every check of one quantised layer; nothing is enqueued
static int validate_linear_q(const void* x, const eora_q_member& e, int M, int d_in, int r, int w_bits, int group,
                             int ab_bits, const void* workspace, size_t workspace_bytes, int* fa, int* fe)
{
    if (!x || !e.qweight || !e.scales || !e.qzeros || !e.y) return EORA_ERR_NULL;
    if (w_bits < 2 || w_bits > 4) return EORA_ERR_UNSUPPORTED;
    int rc = check_backbone_shape(M, d_in, e.d_out, r);
    if (rc != EORA_OK) return rc;
    rc = check_group(d_in, group);
    if (rc != EORA_OK) return rc;
    *fe = *fa = S_NONE;
    if (r > 0) {
        if (!e.A || !e.B) return EORA_ERR_NULL;
        if (ab_bits != 16 && ab_bits != 4 && ab_bits != 3) return EORA_ERR_UNSUPPORTED;
        if (ab_bits != 16 && (!e.A_scales || !e.B_scales)) return EORA_ERR_NULL;
        rc = factor_formats(r, ab_bits, fa, fe);
        if (rc != EORA_OK) return rc;
        if (!aligned16(e.A) || !aligned16(e.B) || !aligned16(e.A_scales) || !aligned16(e.B_scales)) return EORA_ERR_ALIGN;
    }
    if (!aligned16(x) || !aligned16(e.qweight) || !aligned16(e.scales) || !aligned16(e.qzeros) || !aligned16(e.y))
        return EORA_ERR_ALIGN;
    if (!workspace) return EORA_ERR_WORKSPACE;
    if (!aligned16(workspace)) return EORA_ERR_ALIGN;
    if (workspace_bytes < workspace_min_bytes(M, d_in, e.d_out, r)) return EORA_ERR_WORKSPACE;
    return EORA_OK;
}

// one validated quantised layer
static int run_linear_q(const void* x, const eora_q_member& e, int M, int d_in, int r, int w_bits, int group, int ab_bits,
                        int fa, int fe, void* workspace, size_t workspace_bytes, void* stream)
{
    const int d_out = e.d_out;
    if (M == 0) return EORA_OK;

    if (prefill_fits(M, r, ab_bits)) return launch_prefill_group(x, &e, 1, M, d_in, r, w_bits, group, fa, fe, nullptr, 0, workspace, workspace_bytes, (hipStream_t)stream);

    int nw = 0, nq = 0;
    if (small_kernel_fits(M, d_in, group, &nw, &nq))
        return launch_group(x, &e, 1, M, d_in, r, w_bits, group, fa, fe, nw, nq, workspace, (hipStream_t)stream);

    if (stream_fits(M, d_in, group, r, backbone_format(w_bits), fa, &d_out, 1))
        return launch_stream_group(x, &e, 1, M, d_in, r, w_bits, fa, fe, workspace, (hipStream_t)stream);

    return launch_wide_group(x, &e, 1, M, d_in, r, w_bits, group, fa, fe, workspace, workspace_bytes, (hipStream_t)stream);
}

int eora_linear_q(const void* x, const void* qweight, const void* scales, const void* qzeros,
                  const void* A, const void* B, const void* A_scales, const void* B_scales,
                  void* y, int M, int d_in, int d_out, int r, int w_bits, int group, int ab_bits,
                  void* workspace, size_t workspace_bytes, void* stream)
{
    const eora_q_member e{qweight, scales, qzeros, A, B, A_scales, B_scales, y, d_out};
    int fa, fe;
    const int rc = validate_linear_q(x, e, M, d_in, r, w_bits, group, ab_bits, workspace, workspace_bytes, &fa, &fe);
    if (rc != EORA_OK) return rc;
    return run_linear_q(x, e, M, d_in, r, w_bits, group, ab_bits, fa, fe, workspace, workspace_bytes, stream);
}

// ---- the same layer for callers that cannot allocate ---------------------------------------------------------
namespace {
// Workspace of eora_linear_q_static: one array per GPU the library's code is loaded on, held until the process
// ends.  Its size is that of eora_workspace_bytes() for any call below PREFILL_MIN_TOKENS tokens (header, tagged
// partials, fp32 partials).  In host code the array's name is only a handle for hipGetSymbolAddress: the device
// address it yields (per device) is what kernels and the clearing launch are given.
constexpr size_t STATIC_SCRATCH_BYTES = WS_T + WIDE_SPLIT_BYTES;
__device__ __align__(256) unsigned char scratch[STATIC_SCRATCH_BYTES];
constexpr int MAX_DEVICES = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[MAX_DEVICES] = {};
bool g_scratch_cleared[MAX_DEVICES] = {};

// the current device's array, cleared (enqueued on `stream`) the first time it is handed out
int static_scratch(void** out, hipStream_t stream)
{
    int device = -1;
    if (hipGetDevice(&device) != hipSuccess || device < 0 || device >= MAX_DEVICES) return EORA_ERR_LAUNCH;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[device]) {
        void* p = nullptr;
        if (failed(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)), "static scratch address") || !p) return EORA_ERR_LAUNCH;
        g_scratch_ptr[device] = p;
    }
    if (!g_scratch_cleared[device]) {
        const int rc = eora_workspace_init(g_scratch_ptr[device], STATIC_SCRATCH_BYTES, stream);
        if (rc != EORA_OK) return rc;
        g_scratch_cleared[device] = true;
    }
    *out = g_scratch_ptr[device];
    return EORA_OK;
}
}  // namespace

int eora_linear_q_static(const void* x, const void* qweight, const void* scales, const void* qzeros,
                         const void* A, const void* B, const void* A_scales, const void* B_scales,
                         void* y, int M, int d_in, int d_out, int r, int w_bits, int group, int ab_bits, void* stream)
{
    if (M >= PREFILL_MIN_TOKENS) return EORA_ERR_WORKSPACE;       // the many-token path needs scratch that grows with M
    const eora_q_member e{qweight, scales, qzeros, A, B, A_scales, B_scales, y, d_out};
    int fa, fe;
    // every check before the array is touched (a placeholder stands in for the workspace pointer)
    int rc = validate_linear_q(x, e, M, d_in, r, w_bits, group, ab_bits, x, STATIC_SCRATCH_BYTES, &fa, &fe);
    if (rc != EORA_OK) return rc;
    if (M == 0) return EORA_OK;
    void* ws = nullptr;
    rc = static_scratch(&ws, (hipStream_t)stream);
    if (rc != EORA_OK) return rc;
    return run_linear_q(x, e, M, d_in, r, w_bits, group, ab_bits, fa, fe, ws, STATIC_SCRATCH_BYTES, stream);
}

int eora_linear_q_multi(const void* x, const void* qweight, const void* scales, const void* qzeros,
                        const void* A_all, const void* B_all, const void* A_scales, const void* B_scales,
                        const void* adapter_of_row, void* y, int M, int d_in, int d_out, int r, int n_adapters,
                        int w_bits, int group, int ab_bits, void* workspace, size_t workspace_bytes, void* stream)
{
    if (n_adapters < 1 || r < 1 || r % 32 || (ab_bits != 16 && r % 128)) return EORA_ERR_SHAPE;
    if ((long long)n_adapters * r > MAX_RANK) return EORA_ERR_SHAPE;
    if (!adapter_of_row) return EORA_ERR_NULL;
    if (reinterpret_cast<uintptr_t>(adapter_of_row) & 3u) return EORA_ERR_ALIGN;
    const int R = n_adapters * r;
    const eora_q_member e{qweight, scales, qzeros, A_all, B_all, A_scales, B_scales, y, d_out};
    int fa, fe;
    const int rc = validate_linear_q(x, e, M, d_in, R, w_bits, group, ab_bits, workspace, workspace_bytes, &fa, &fe);
    if (rc != EORA_OK) return rc;
    if (M == 0) return EORA_OK;
    // many tokens: the GEMM path, with t masked per row between its two launches
    if (prefill_fits(M, R, ab_bits))
        return launch_prefill_group(x, &e, 1, M, d_in, R, w_bits, group, fa, fe, (const int*)adapter_of_row, r, workspace, workspace_bytes, (hipStream_t)stream);
    // one to four tokens: the decode kernel, with t masked where it is gathered
    int nw = 0, nq = 0;
    if (small_kernel_fits(M, d_in, group, &nw, &nq))
        return launch_group(x, &e, 1, M, d_in, R, w_bits, group, fa, fe, nw, nq, workspace, (hipStream_t)stream, (const int*)adapter_of_row, r);
    // 5 .. 16 tokens and enough rows: the kernel with x resident in LDS, with t masked where it goes to LDS
    if (stream_fits(M, d_in, group, R, backbone_format(w_bits), fa, &d_out, 1))
        return launch_stream_group(x, &e, 1, M, d_in, R, w_bits, fa, fe, workspace, (hipStream_t)stream, (const int*)adapter_of_row, r);
    return launch_wide_group(x, &e, 1, M, d_in, R, w_bits, group, fa, fe, workspace, workspace_bytes, (hipStream_t)stream, (const int*)adapter_of_row, r);
}

int eora_linear_q_group(const void* x, const eora_q_member* members, int n_members,
                        int M, int d_in, int r, int w_bits, int group, int ab_bits,
                        void* workspace, size_t workspace_bytes, void* stream)
{
    if (!x || !members) return EORA_ERR_NULL;
    if (n_members < 1 || n_members > MAX_GROUP) return EORA_ERR_SHAPE;
    int fa = S_NONE, fe = S_NONE;
    for (int m = 0; m < n_members; ++m) {               // every member is validated before anything is enqueued
        const int rc = validate_linear_q(x, members[m], M, d_in, r, w_bits, group, ab_bits, workspace, workspace_bytes, &fa, &fe);
        if (rc != EORA_OK) return rc;
    }
    int nw = 0, nq = 0;
    // one to four tokens: every group of shapes the decode kernel takes (it hands t over in tagged pairs alone, without the
    // header's flags; four members of rank 512 in four ranges fill half of the pairs' region)
    if (small_kernel_fits(M, d_in, group, &nw, &nq))
        return launch_group(x, members, n_members, M, d_in, r, w_bits, group, fa, fe, nw, nq, workspace, (hipStream_t)stream);
    if (prefill_fits(M, r, ab_bits) && workspace_bytes >= workspace_group_min_bytes(M, d_in, r, n_members))
        return launch_prefill_group(x, members, n_members, M, d_in, r, w_bits, group, fa, fe, nullptr, 0, workspace, workspace_bytes, (hipStream_t)stream);
    if (n_members >= 1) {
        int rows[MAX_GROUP] = {0, 0, 0, 0};
        for (int m = 0; m < n_members; ++m) rows[m] = members[m].d_out;
        if (stream_fits(M, d_in, group, r, backbone_format(w_bits), fa, rows, n_members))
            return launch_stream_group(x, members, n_members, M, d_in, r, w_bits, fa, fe, workspace, (hipStream_t)stream);
    }
    // one launch of the general kernel, as long as the members' t fits its region (64 tokens per group of token blocks)
    if (n_members > 1 && M > 0 && !prefill_fits(M, r, ab_bits) &&
        (size_t)n_members * (((M < CHUNK_TOKENS ? M : CHUNK_TOKENS) + 63) / 64) * 64 * r <= MAX_PART_ELEMS)
        return launch_wide_group(x, members, n_members, M, d_in, r, w_bits, group, fa, fe, workspace, workspace_bytes, (hipStream_t)stream);
    for (int m = 0; m < n_members; ++m) {               // other shapes (or a workspace sized for one member): one after the other
        const int rc = run_linear_q(x, members[m], M, d_in, r, w_bits, group, ab_bits, fa, fe, workspace, workspace_bytes, stream);
        if (rc != EORA_OK) return rc;
    }
    return EORA_OK;
}

namespace {
// both 2:4 entry points: exactly one of values / qvalues is given
int run_linear_sparse(const void* x, const void* values, const void* indices, const void* qtiles, const void* qmeta,
                      const void* A, const void* B, void* y,
                      int M, int d_in, int d_out, int r, void* workspace, size_t workspace_bytes, void* stream)
{
    int rc = check_backbone_shape(M, d_in, d_out, r);
    if (rc != EORA_OK) return rc;
    if (r > 0) {
        if (!A || !B) return EORA_ERR_NULL;
        if (r % 32) return EORA_ERR_SHAPE;
        if (!aligned16(A) || !aligned16(B)) return EORA_ERR_ALIGN;
    }
    if (!aligned16(x) || !aligned16(values) || !aligned16(qtiles) || !aligned16(qmeta) || !aligned16(indices) || !aligned16(y)) return EORA_ERR_ALIGN;
    if (!workspace) return EORA_ERR_WORKSPACE;
    if (!aligned16(workspace)) return EORA_ERR_ALIGN;
    if (workspace_bytes < workspace_min_bytes(M, d_in, d_out, r)) return EORA_ERR_WORKSPACE;
    if (M == 0) return EORA_OK;
    int kcn = pick_kcn(M, d_in);
    // (the longest contractions at 1..4 tokens: sixteen ranges, so that the producers are done before the first
    // consumers reach their tails; 70B down projection 51.1 -> 50.4 us, with 4-bit kept values 29.5 -> 27.7 us)
    if (M <= 4 && d_in > 16384 && (d_in / 128) % 16 == 0 && (r / 16) * 16 <= HDR_FLAGS_PER_BLOCK) kcn = 16;
    for (int m0 = 0; m0 < M; m0 += CHUNK_TOKENS) {
        SparseArgs a{};
        a.x = (const _Float16*)x + (size_t)m0 * d_in;
        a.values = (const _Float16*)values;
        a.indices = (const uint32_t*)indices;
        a.qtiles = (const uint32_t*)qtiles;
        a.qmeta = (const uint32_t*)qmeta;
        a.A = A;
        a.B = B;
        a.y = (_Float16*)y + (size_t)m0 * d_out;
        a.hdr = (uint32_t*)workspace;
        a.tpart = (float*)((char*)workspace + WS_PARTS);
        a.tpair = (unsigned long long*)((char*)workspace + WS_PAIRS);
        a.M = M - m0 < CHUNK_TOKENS ? M - m0 : CHUNK_TOKENS;
        a.d_in = d_in;
        a.d_out = d_out;
        a.r = r;
        a.kcn = kcn;
        a.spin_limit = g_spin_limit;
        a.ksplit = 1;
        a.ypart = sparse_split_bytes(M, d_in, d_out) ? (float*)((char*)workspace + WS_T) : nullptr;
        if (failed(launch_sparse(a, (hipStream_t)stream), "linear_sp24")) return EORA_ERR_LAUNCH;
    }
    return EORA_OK;
}
}  // namespace

int eora_linear_sp24_group(const void* x, const eora_sp_member* members, int n_members,
                           int M, int d_in, int r, void* workspace, size_t workspace_bytes, void* stream)
{
    if (!x || !members) return EORA_ERR_NULL;
    if (n_members < 1 || n_members > MAX_GROUP) return EORA_ERR_SHAPE;
    const bool vq = members[0].qtiles != nullptr;
    for (int m = 0; m < n_members; ++m) {               // every member is validated before anything is enqueued
        const eora_sp_member& e = members[m];
        if (!e.y) return EORA_ERR_NULL;
        if (vq ? (!e.qtiles || !e.qmeta || e.values || e.indices) : (!e.values || !e.indices || e.qtiles || e.qmeta)) return EORA_ERR_NULL;
        int rc = check_backbone_shape(M, d_in, e.d_out, r);
        if (rc != EORA_OK) return rc;
        if (r > 0) {
            if (!e.A || !e.B) return EORA_ERR_NULL;
            if (r % 32) return EORA_ERR_SHAPE;
            if (!aligned16(e.A) || !aligned16(e.B)) return EORA_ERR_ALIGN;
        }
        if (!aligned16(x) || !aligned16(e.values) || !aligned16(e.qtiles) || !aligned16(e.qmeta) || !aligned16(e.indices) || !aligned16(e.y))
            return EORA_ERR_ALIGN;
        if (!workspace) return EORA_ERR_WORKSPACE;
        if (!aligned16(workspace)) return EORA_ERR_ALIGN;
        if (workspace_bytes < workspace_min_bytes(M, d_in, e.d_out, r)) return EORA_ERR_WORKSPACE;
    }
    if (M == 0) return EORA_OK;
    // one launch when the members' partials and flags fit the regions of one call; else one after the other
    const int yblocks = (M + 15) / 16;
    int kcn = pick_kcn(M, d_in);
    // (the longest contractions at 1..4 tokens: sixteen ranges, so that the producers are done before the first
    // consumers reach their tails; 70B down projection 51.1 -> 50.4 us, with 4-bit kept values 29.5 -> 27.7 us)
    if (M <= 4 && d_in > 16384 && (d_in / 128) % 16 == 0 && (r / 16) * 16 <= HDR_FLAGS_PER_BLOCK) kcn = 16;
    while (kcn > 1 && (n_members * yblocks * kcn > 32 || (d_in / 128) % kcn)) --kcn;
    const bool one_launch = n_members > 1 && M <= CHUNK_TOKENS && n_members * yblocks * kcn <= 32 &&
                            (r / 16) * kcn * n_members <= HDR_FLAGS_PER_BLOCK;
    if (!one_launch) {
        for (int m = 0; m < n_members; ++m) {
            const eora_sp_member& e = members[m];
            const int rc = run_linear_sparse(x, e.values, e.indices, e.qtiles, e.qmeta, e.A, e.B, e.y, M, d_in, e.d_out, r,
                                             workspace, workspace_bytes, stream);
            if (rc != EORA_OK) return rc;
        }
        return EORA_OK;
    }
    SparseArgs as[MAX_GROUP];
    for (int m = 0; m < n_members; ++m) {
        const eora_sp_member& e = members[m];
        SparseArgs a{};
        a.x = (const _Float16*)x;
        a.values = (const _Float16*)e.values;
        a.indices = (const uint32_t*)e.indices;
        a.qtiles = (const uint32_t*)e.qtiles;
        a.qmeta = (const uint32_t*)e.qmeta;
        a.A = e.A;
        a.B = e.B;
        a.y = (_Float16*)e.y;
        a.hdr = (uint32_t*)workspace;
        const size_t region = (size_t)m * yblocks * kcn * 16 * r;        // this member's partials of t
        a.tpart = (float*)((char*)workspace + WS_PARTS) + region;
        a.tpair = (unsigned long long*)((char*)workspace + WS_PAIRS) + region;
        a.M = M;
        a.d_in = d_in;
        a.d_out = e.d_out;
        a.r = r;
        a.kcn = kcn;
        a.spin_limit = g_spin_limit;
        a.ksplit = 1;                                                    // (grouped launches never split the contraction)
        as[m] = a;
    }
    if (failed(launch_sparse_group(as, n_members, (hipStream_t)stream), "linear_sp24_group")) return EORA_ERR_LAUNCH;
    return EORA_OK;
}

int eora_linear_sp24(const void* x, const void* values, const void* indices,
                     const void* A, const void* B, void* y,
                     int M, int d_in, int d_out, int r,
                     void* workspace, size_t workspace_bytes, void* stream)
{
    if (!x || !values || !indices || !y) return EORA_ERR_NULL;
    return run_linear_sparse(x, values, indices, nullptr, nullptr, A, B, y, M, d_in, d_out, r,
                             workspace, workspace_bytes, stream);
}

int eora_linear_sp24q4(const void* x, const void* qtiles, const void* qmeta,
                       const void* A, const void* B, void* y,
                       int M, int d_in, int d_out, int r,
                       void* workspace, size_t workspace_bytes, void* stream)
{
    if (!x || !qtiles || !qmeta || !y) return EORA_ERR_NULL;
    return run_linear_sparse(x, nullptr, nullptr, qtiles, qmeta, A, B, y, M, d_in, d_out, r,
                             workspace, workspace_bytes, stream);
}

int eora_unpack_q(const void* qweight, const void* qzeros, void* codes_u8, void* zeros_u8,
                  int d_in, int d_out, int w_bits, int group, void* stream)
{
    if (!qweight || !qzeros || !codes_u8 || !zeros_u8) return EORA_ERR_NULL;
    if (w_bits < 2 || w_bits > 4) return EORA_ERR_UNSUPPORTED;
    int rc = check_backbone_shape(1, d_in, d_out, 0);
    if (rc != EORA_OK) return rc;
    rc = check_group(d_in, group);
    if (rc != EORA_OK) return rc;
    if (!aligned16(qweight) || !aligned16(qzeros)) return EORA_ERR_ALIGN;
    if (failed(launch_unpack_q((const uint32_t*)qweight, (const uint32_t*)qzeros, (uint8_t*)codes_u8,
                               (uint8_t*)zeros_u8, d_in, d_out, w_bits, group, (hipStream_t)stream), "unpack_q"))
        return EORA_ERR_LAUNCH;
    return EORA_OK;
}

int eora_dequant_q(const void* qweight, const void* scales, const void* qzeros, void* W_f32,
                   int d_in, int d_out, int w_bits, int group, void* stream)
{
    if (!qweight || !scales || !qzeros || !W_f32) return EORA_ERR_NULL;
    if (w_bits < 2 || w_bits > 4) return EORA_ERR_UNSUPPORTED;
    int rc = check_backbone_shape(1, d_in, d_out, 0);
    if (rc != EORA_OK) return rc;
    rc = check_group(d_in, group);
    if (rc != EORA_OK) return rc;
    if (!aligned16(qweight) || !aligned16(scales) || !aligned16(qzeros) || !aligned16(W_f32)) return EORA_ERR_ALIGN;
    if (failed(launch_dequant_q((const uint32_t*)qweight, (const _Float16*)scales, (const uint32_t*)qzeros,
                                (float*)W_f32, d_in, d_out, w_bits, group, (hipStream_t)stream), "dequant_q"))
        return EORA_ERR_LAUNCH;
    return EORA_OK;
}

int eora_expand_sp24(const void* values, const void* indices, void* W_f16, int d_in, int d_out, void* stream)
{
    if (!values || !indices || !W_f16) return EORA_ERR_NULL;
    int rc = check_backbone_shape(1, d_in, d_out, 0);
    if (rc != EORA_OK) return rc;
    if (!aligned16(values) || !aligned16(indices) || !aligned16(W_f16)) return EORA_ERR_ALIGN;
    if (failed(launch_expand_sp24((const _Float16*)values, (const uint32_t*)indices, (_Float16*)W_f16, d_in, d_out,
                                  (hipStream_t)stream), "expand_sp24"))
        return EORA_ERR_LAUNCH;
    return EORA_OK;
}

int eora_expand_sp24q4(const void* qtiles, const void* qmeta, void* W_f32, int d_in, int d_out, void* stream)
{
    if (!qtiles || !qmeta || !W_f32) return EORA_ERR_NULL;
    int rc = check_backbone_shape(1, d_in, d_out, 0);
    if (rc != EORA_OK) return rc;
    if (!aligned16(qtiles) || !aligned16(qmeta) || !aligned16(W_f32)) return EORA_ERR_ALIGN;
    if (failed(launch_expand_sp24q4((const uint32_t*)qtiles, (const uint32_t*)qmeta, (float*)W_f32, d_in, d_out,
                                    (hipStream_t)stream), "expand_sp24q4"))
        return EORA_ERR_LAUNCH;
    return EORA_OK;
}

}  // extern "C"
