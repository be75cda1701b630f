// Algorithm 1 (Sec. 3), steps 1-6, in fp64 on the device: the factors B' (d_out x r) and A (r x d_in) that
// compensate a compressed weight, from the weight, its compressed version and calibration activations.
//
//   1  dW = W - What
//   2  X~ X~^T = Q Lambda Q^T          one-sided Jacobi on the rows of the Gram matrix (rotations accumulated)
//   3  Q' = Q sqrt(Lambda)
//   4  dW' = dW Q'
//   5  rank-r SVD of dW'               one-sided Jacobi on the rows of dW' (or of its transpose, whichever
//                                      has fewer rows), top r rows by norm
//   6  A = A' sqrt(Lambda)^-1 Q^T
//
// One-sided (Hestenes) Jacobi: plane rotations of row pairs until all rows are mutually orthogonal.  For a
// symmetric positive semi-definite G, R G with orthogonal rows means R G^2 R^T is diagonal, so the rows of the
// accumulated rotation R are eigenvectors of G and r_p . (R G)_p its eigenvalues.  For a general matrix T,
// R T with orthogonal rows is Sigma V^T (row norms = singular values, R = U^T).  A round of the round-robin
// schedule rotates m/2 disjoint pairs, one workgroup per pair, rows held in registers; m-1 rounds visit every
// pair once (a sweep); sweeps repeat until one passes whose rotations, if any, were all so small that nothing is left after them (NEARLY below).
#include "eora.h"

#include <hip/hip_runtime.h>
#include <cmath>
#include <type_traits>
#include <cstdint>
#include <cstdio>
#include <cstdlib>

namespace eora {
namespace {

constexpr int JPT = 8;                 // double2 items per thread and row
constexpr int MAX_DIM = 16384;         // 2 * JPT * 1024
constexpr int MAX_SWEEPS = 60;

__device__ inline double wave_sum(double v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// What became of the pairs of a workgroup: none was to be rotated; all that were had a sine and a cosine between the rows of at most
// `small`; others.  A sweep rotates every pair once.  A later rotation of one of its rows puts a sine times a cosine back into a pair's own
// cosine, times the ratio of the two rotated rows' norms where the other one is larger: at most 1.62 small^2, as a large ratio makes the sine of
// a given cosine small (s = c rho / (rho^2 - 1), both at the limit at rho = 1.62).  There are 2 m of them: with small = sqrt(tol / 4 m) they leave
// 0.81 tol of a pair that was rotated, and 1.81 tol of one that was just below tol and left alone.  A sweep without ROTATED is therefore the last one and
// needs no other to find that nothing is left (4096 x 4096, rank 128: 31.3 -> 30.7 ms; 2048 x 2048, rank 256: 31.0 -> 29.4; left in tests: 1.0 tol).
enum { ORTHOGONAL = 0, NEARLY = 1, ROTATED = 2 };

// Every workgroup of a round counts in a word of its own: rounds in which it rotated rows in the low half, those of them with a rotation that was
// not small in the high half.  One word for all makes a round's additions come one after the other, at its end: a round over 578 rows (289 workgroups) takes 4.5 us
// so, 6.1 with one word; 640 x 578, rank 224 50.5 -> 36.6 ms, 300 x 300 18.8 -> 15.4.
__device__ __forceinline__ void count_rotation(unsigned long long* mine, int turned)
{
    atomicAdd(mine, turned == ROTATED ? 0x100000001ull : 1ull);
}

// One round: workgroup i rotates the row pair (p, q) of the round-robin schedule.  H: m x L row-major;
// V: m x m row-major or nullptr.  rows with squared norm <= abs_floor count as zero.
template <int NT>
__global__ __launch_bounds__(NT) void jacobi_round_kernel(double* __restrict__ H, int L, double* __restrict__ V,
                                                          int m, int round, double tol, double abs_floor, double small,
                                                          unsigned long long* __restrict__ rotations)
{
    const int i = blockIdx.x, mm = m - 1, tid = threadIdx.x;
    int p, q;
    if (i == 0) {
        p = round;
        q = mm;
    } else {
        p = (round + i) % mm;
        q = (round + mm - i) % mm;
    }
    const int L2 = L >> 1;
    double2* rp = reinterpret_cast<double2*>(H + (size_t)p * L);
    double2* rq = reinterpret_cast<double2*>(H + (size_t)q * L);
    double2 hp[JPT], hq[JPT];
    double app = 0, aqq = 0, apq = 0;
#pragma unroll
    for (int k = 0; k < JPT; ++k) {
        const int idx = tid + k * NT;
        hp[k] = hq[k] = make_double2(0.0, 0.0);
        if (idx < L2) {
            hp[k] = rp[idx];
            hq[k] = rq[idx];
        }
        app += hp[k].x * hp[k].x + hp[k].y * hp[k].y;
        aqq += hq[k].x * hq[k].x + hq[k].y * hq[k].y;
        apq += hp[k].x * hq[k].x + hp[k].y * hq[k].y;
    }
    __shared__ double red[3][16];
    __shared__ double cs[2];
    __shared__ int go;
    app = wave_sum(app);
    aqq = wave_sum(aqq);
    apq = wave_sum(apq);
    constexpr int NWV = NT / 64;
    if ((tid & 63) == 0) {
        red[0][tid >> 6] = app;
        red[1][tid >> 6] = aqq;
        red[2][tid >> 6] = apq;
    }
    __syncthreads();
    if (tid == 0) {
        double a = 0, b = 0, c = 0;
        for (int w = 0; w < NWV; ++w) {
            a += red[0][w];
            b += red[1][w];
            c += red[2][w];
        }
        int rotate = ORTHOGONAL;
        if (a > abs_floor && b > abs_floor && fabs(c) > tol * sqrt(a) * sqrt(b)) {
            const double zeta = (b - a) / (2.0 * c);
            const double t = copysign(1.0, zeta) / (fabs(zeta) + sqrt(1.0 + zeta * zeta));
            const double co = 1.0 / sqrt(1.0 + t * t);
            cs[0] = co;
            cs[1] = co * t;
            rotate = fabs(co * t) <= small && fabs(c) <= small * sqrt(a) * sqrt(b) ? NEARLY : ROTATED;
        }
        go = rotate;
    }
    __syncthreads();
    if (go == ORTHOGONAL) return;
    if (tid == 0) count_rotation(rotations + i, go);
    const double co = cs[0], si = cs[1];
#pragma unroll
    for (int k = 0; k < JPT; ++k) {
        const int idx = tid + k * NT;
        if (idx < L2) {
            rp[idx] = make_double2(co * hp[k].x - si * hq[k].x, co * hp[k].y - si * hq[k].y);
            rq[idx] = make_double2(si * hp[k].x + co * hq[k].x, si * hp[k].y + co * hq[k].y);
        }
    }
    if (V) {
        double2* vp = reinterpret_cast<double2*>(V + (size_t)p * m);
        double2* vq = reinterpret_cast<double2*>(V + (size_t)q * m);
        for (int idx = tid; idx < (m >> 1); idx += NT) {
            const double2 a = vp[idx], b = vq[idx];
            vp[idx] = make_double2(co * a.x - si * b.x, co * a.y - si * b.y);
            vq[idx] = make_double2(si * a.x + co * b.x, si * a.y + co * b.y);
        }
    }
}

// ------------------------------------------------------------------------------------------------------------
// Block version of a round, for m % 16 == 0 and row lengths that are multiples of 128: a workgroup takes two
// blocks of eight rows (16 x L), forms their 16 x 16 Gram matrix S with fp64 MFMAs, diagonalises S in LDS with a
// small two-sided Jacobi iteration (S = J D J^T, J orthogonal), and replaces the rows by J^T times the rows
// (MFMAs again), which makes all 16 mutually orthogonal at once: 120 row pairs for three passes over the rows
// instead of one pair for two.  The eigenvector rows get the same J^T.
//
// v_mfma_f64_16x16x4_f64 operand layout (lane l, n = l % 16, g = l / 16): A[i = n][k = g], B[k = g][j = n],
// result register v holds D[i = 4 v + g][j = n].
typedef double d4 __attribute__((ext_vector_type(4)));
constexpr int BJ_NT = 512, BJ_NW = BJ_NT / 64;
__device__ __forceinline__ d4 mfma64(double a, double b, d4 c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }

__device__ __forceinline__ double rcp_approx(double v) { return __builtin_amdgcn_rcp(v); }
__device__ __forceinline__ double rsq_approx(double v) { return __builtin_amdgcn_rsq(v); }

// 1 / sqrt(v) to the last bits but one: two Newton steps on the machine's approximation
__device__ __forceinline__ double rsq_newton(double v)
{
    double y = rsq_approx(v);
#pragma unroll
    for (int i = 0; i < 2; ++i) y = fma(0.5 * y, fma(-v * y, y, 1.0), y);
    return y;
}

// Cosine and sine of the plane rotation that makes [a c; c b] diagonal.  The steps of a 16 x 16 matrix are a chain in which
// each waits for these values, and the library's division and square root are some 30 dependent instructions each.  The
// angle may be off in its last bits (what it leaves of c the next sweep finds), the rotation may not: cosine and sine come
// from one t, so their squares add to 1 to rounding whatever t is.
__device__ __forceinline__ void jacobi_angle(double a, double b, double c, double& co, double& si)
{
    const double d = b - a, h = c + c, rh = rcp_approx(h), q0 = d * rh;
    const double zeta = fma(fma(-h, q0, d), rh, q0);
    const double az = fmin(fabs(zeta), 1e100);            // (c that is next to nothing: no infinities further on)
    const double w = fma(az, az, 1.0), root = w * rsq_approx(w);
    double t = rcp_approx(az + root);                     // the smaller root of t^2 + 2 |zeta| t - 1
    t = fma(-fma(t, t + 2.0 * az, -1.0), 0.5 * rcp_approx(t + az), t);
    t = copysign(t, zeta);
    co = rsq_newton(fma(t, t, 1.0));
    si = co * t;
}

// value of lane `from` (4 times its number) in every lane
__device__ __forceinline__ double lane_value(double v, int from4)
{
    const unsigned long long u = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = (unsigned)__builtin_amdgcn_ds_bpermute(from4, (int)(unsigned)u);
    const unsigned hi = (unsigned)__builtin_amdgcn_ds_bpermute(from4, (int)(unsigned)(u >> 32));
    return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

// Whether a pair of rows with squared norms a, b and product c is to be rotated
__device__ __forceinline__ bool rotation_due(double a, double b, double c, double tol, double abs_floor)
{
    return a > abs_floor && b > abs_floor && fabs(c) > tol * (a * rsq_approx(a)) * (b * rsq_approx(b));
}

__device__ __forceinline__ bool rotation_large(double a, double b, double c, double si, double small)
{
    return !(fabs(si) <= small) || !(fabs(c) <= small * (a * rsq_approx(a)) * (b * rsq_approx(b)));
}

// S (Gram matrix of 16 rows: a block of eight, P, and another, Q) -> J orthogonal, after one rotation of each of the 64 pairs of a
// row of P and a row of Q, in eight steps of eight disjoint pairs (i, (i + step) mod 8).  One wavefront.
// Lane (i, j) holds the 2 x 2 block of S in the rows of pair i and the columns of pair j, and rows 2 i, 2 i + 1 of J's columns of
// pair j.  From one step to the next P's places stay and Q's move up by one lane of their index, so the matrix never leaves the
// registers; the eight lanes (i, i) find the angles, every lane fetches those of its two pairs.  (Through LDS, with every lane
// forming its two angles, a step took 1270 cycles, and a round of rows took all 120 pairs in 15 steps: those within P and within Q
// belong to one round of a sweep.)
__device__ __forceinline__ int rotate_cross_pairs(const double (*S)[17], double (*J)[17], int lane, double tol, double abs_floor, double small)
{
    const int i = lane >> 3, j = lane & 7;
    if (!__any(rotation_due(S[i][i], S[8 + j][8 + j], S[i][8 + j], tol, abs_floor))) return ORTHOGONAL;
    bool large = false;
    double pp = S[i][j], pq = S[i][8 + j], qp = S[8 + i][j], qq = S[8 + i][8 + j];
    double jp0 = 2 * i == j ? 1.0 : 0.0, jp1 = 2 * i + 1 == j ? 1.0 : 0.0, jq0 = 2 * i == 8 + j ? 1.0 : 0.0, jq1 = 2 * i + 1 == 8 + j ? 1.0 : 0.0;
    const int row = 4 * 9 * i, col = 4 * 9 * j;           // lanes (i, i) and (j, j)
    const int nr = 4 * (8 * ((i + 1) & 7) + j), nc = 4 * (8 * i + ((j + 1) & 7)), nrc = 4 * (8 * ((i + 1) & 7) + ((j + 1) & 7));
#pragma unroll 1
    for (int step = 0; step < 8; ++step) {
        double co, si;
        jacobi_angle(pp, qq, pq, co, si);
        const bool on = rotation_due(pp, qq, pq, tol, abs_floor);      // (of lanes (i, i); the others' are nobody's)
        large = large || (i == j && on && rotation_large(pp, qq, pq, si, small));
        co = on ? co : 1.0;
        si = on ? si : 0.0;
        const double co0 = lane_value(co, row), si0 = lane_value(si, row), co1 = lane_value(co, col), si1 = lane_value(si, col);
        const double tpp = co0 * pp - si0 * qp, tqp = si0 * pp + co0 * qp;      // rows
        const double tpq = co0 * pq - si0 * qq, tqq = si0 * pq + co0 * qq;
        pp = co1 * tpp - si1 * tpq;                                             // columns
        pq = lane_value(si1 * tpp + co1 * tpq, nc);
        qp = lane_value(co1 * tqp - si1 * tqq, nr);
        qq = lane_value(si1 * tqp + co1 * tqq, nrc);
        const double n0 = si1 * jp0 + co1 * jq0, n1 = si1 * jp1 + co1 * jq1;
        jp0 = co1 * jp0 - si1 * jq0;
        jp1 = co1 * jp1 - si1 * jq1;
        jq0 = lane_value(n0, nc);
        jq1 = lane_value(n1, nc);
    }
    J[2 * i][j] = jp0;
    J[2 * i + 1][j] = jp1;
    J[2 * i][8 + j] = jq0;
    J[2 * i + 1][8 + j] = jq1;
    return __any(large) ? ROTATED : NEARLY;
}

// The same for all 120 pairs of the 16 rows, in fifteen steps of eight: the rounds that also see to the pairs within a block.
// Lane (i, j) owns the 2 x 2 block of S in the rows of pair i and the columns of pair j, forms both pairs' rotations by
// itself and applies them from either side at once, and turns rows 2 i, 2 i + 1 of J's columns of pair j: one round through
// LDS per step (one wavefront's LDS operations are carried out in order).
__device__ __forceinline__ int rotate_all_pairs(double (*S)[17], double (*J)[17], int lane, double tol, double abs_floor, double small)
{
    const int pi = lane >> 3, pj = lane & 7;
    bool some = false;                                // whether any of the 120 pairs is to be rotated (in the last sweeps most rounds have none)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int r = (lane >> 4) + 4 * e, c = lane & 15;
        some = some || (r < c && rotation_due(S[r][r], S[c][c], S[r][c], tol, abs_floor));
        J[r][c] = r == c ? 1.0 : 0.0;
    }
    if (!__any(some)) return ORTHOGONAL;
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    bool any = false, large = false;
#pragma unroll 1
    for (int step = 0; step < 15; ++step) {
        auto pair = [&](int t, int& p, int& q) {
            p = t == 0 ? step : step + t >= 15 ? step + t - 15 : step + t;
            q = t == 0 ? 15 : step + 15 - t >= 15 ? step - t : step + 15 - t;
        };
        int p0, q0, p1, q1;
        pair(pi, p0, q0);
        pair(pj, p1, q1);
        const double a0 = S[p0][p0], b0 = S[q0][q0], c0 = S[p0][q0], a1 = S[p1][p1], b1 = S[q1][q1], c1 = S[p1][q1];
        const double spp = S[p0][p1], spq = S[p0][q1], sqp = S[q0][p1], sqq = S[q0][q1];
        const double jp0 = J[2 * pi][p1], jq0 = J[2 * pi][q1], jp1 = J[2 * pi + 1][p1], jq1 = J[2 * pi + 1][q1];
        double co0, si0, co1, si1;
        jacobi_angle(a0, b0, c0, co0, si0);
        jacobi_angle(a1, b1, c1, co1, si1);
        const bool on0 = rotation_due(a0, b0, c0, tol, abs_floor), on1 = rotation_due(a1, b1, c1, tol, abs_floor);
        large = large || (on1 && rotation_large(a1, b1, c1, si1, small));
        co0 = on0 ? co0 : 1.0;
        si0 = on0 ? si0 : 0.0;
        co1 = on1 ? co1 : 1.0;
        si1 = on1 ? si1 : 0.0;
        if (!__any(on1)) continue;                    // uniform: nothing to rotate in this step
        any = true;
        const double tpp = co0 * spp - si0 * sqp, tqp = si0 * spp + co0 * sqp;      // rows
        const double tpq = co0 * spq - si0 * sqq, tqq = si0 * spq + co0 * sqq;
        S[p0][p1] = co1 * tpp - si1 * tpq;                                          // columns
        S[p0][q1] = si1 * tpp + co1 * tpq;
        S[q0][p1] = co1 * tqp - si1 * tqq;
        S[q0][q1] = si1 * tqp + co1 * tqq;
        J[2 * pi][p1] = co1 * jp0 - si1 * jq0;
        J[2 * pi][q1] = si1 * jp0 + co1 * jq0;
        J[2 * pi + 1][p1] = co1 * jp1 - si1 * jq1;
        J[2 * pi + 1][q1] = si1 * jp1 + co1 * jq1;
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    }
    return !any ? ORTHOGONAL : __any(large) ? ROTATED : NEARLY;
}

// The two blocks of eight rows of workgroup i in round `round` of nb / 2 (round-robin over nb blocks)
__device__ __forceinline__ void block_pair(int i, int round, int nb, int& P, int& Q)
{
    const int mm = nb - 1;
    P = i == 0 ? round : (round + i) % mm;
    Q = i == 0 ? mm : (round + mm - i) % mm;
}

// rows <- J^T rows for the 16 rows (block P, block Q) of X (row length len, a multiple of 128)
__device__ __forceinline__ void apply_rotation(double* __restrict__ X, int len, int P, int Q, const double (*J)[17], int wave,
                                               int lane)
{
    const int n = lane & 15, g = lane >> 4;
    double aJ[4];                       // A operand of step kk: (J^T)[i = n][k = 4 kk + g] = J[4 kk + g][n]
    size_t rowoff[4];                   // rows 4 kk + g (loads) = rows 4 v + g (stores)
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
        const int j = 4 * kk + g;
        aJ[kk] = J[j][n];
        rowoff[kk] = (size_t)(j < 8 ? 8 * P + j : 8 * Q + j - 8) * len;
    }
    const int ngroups = len / 128;      // a group: 128 columns = four chunks of 32 (two columns per lane)
    for (int gi = wave; gi < ngroups; gi += BJ_NW) {
        double2 ld[4][4];
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int kk = 0; kk < 4; ++kk)
                ld[u][kk] = *reinterpret_cast<const double2*>(X + rowoff[kk] + 128 * gi + 32 * u + 2 * n);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            d4 d0 = {0, 0, 0, 0}, d1 = {0, 0, 0, 0};
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) {
                d0 = mfma64(aJ[kk], ld[u][kk].x, d0);
                d1 = mfma64(aJ[kk], ld[u][kk].y, d1);
            }
#pragma unroll
            for (int v = 0; v < 4; ++v)
                *reinterpret_cast<double2*>(X + rowoff[v] + 128 * gi + 32 * u + 2 * n) = make_double2(d0[v], d1[v]);
        }
    }
}

__global__ __launch_bounds__(BJ_NT) void jacobi_block_round_kernel(double* __restrict__ H, int L, double* __restrict__ V, int m,
                                                                    int round, double tol, double abs_floor, double small,
                                                                    unsigned long long* __restrict__ rotations)
{
    __shared__ double Sw[BJ_NW][16][17];
    __shared__ double S[16][17], J[16][17];
    __shared__ int s_rotated;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int n = lane & 15, g = lane >> 4;
    int P, Q;
    block_pair(blockIdx.x, round, m / 8, P, Q);
    // ---- Gram matrix of the 16 rows: lane (n, g) feeds row n, both operands of the MFMA are the same register
    {
        const double* row = H + (size_t)(n < 8 ? 8 * P + n : 8 * Q + n - 8) * L;
        d4 acc = {0, 0, 0, 0};
        const int ngroups = L / 128;
        for (int gi = wave; gi < ngroups; gi += BJ_NW) {
            double2 ld[16];             // columns 128 gi + 8 e + 2 g + {0, 1}, e = 0 .. 15
#pragma unroll
            for (int e = 0; e < 16; ++e) ld[e] = *reinterpret_cast<const double2*>(row + 128 * gi + 8 * e + 2 * g);
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                acc = mfma64(ld[e].x, ld[e].x, acc);
                acc = mfma64(ld[e].y, ld[e].y, acc);
            }
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) Sw[wave][4 * v + g][n] = acc[v];
    }
    __syncthreads();
    if (tid < 256) {
        const int r = tid >> 4, c = tid & 15;
        double t = 0;
#pragma unroll
        for (int w = 0; w < BJ_NW; ++w) t += Sw[w][r][c];
        S[r][c] = t;
    }
    __syncthreads();
    // ---- by one wavefront alone (three workgroup barriers per step cost more than they shared out)
    if (wave == 0) {
        const int turned = round == 0 ? rotate_all_pairs(S, J, lane, tol, abs_floor, small) : rotate_cross_pairs(S, J, lane, tol, abs_floor, small);
        if (lane == 0) s_rotated = turned;
    }
    __syncthreads();
    if (s_rotated == ORTHOGONAL) return;               // the 16 rows were orthogonal already (uniform over the workgroup)
    if (tid == 0) count_rotation(rotations + blockIdx.x, s_rotated);
    apply_rotation(H, L, P, Q, J, wave, lane);
    if (V) apply_rotation(V, m, P, Q, J, wave, lane);
}

// A round over rows of 8 CW values (the Ritz matrices of the subspace iteration), without eigenvector rows.  A chain of latencies:
// a wavefront's CW columns of the 16 rows are requested twice, as the operands of the Gram matrix and as those of the
// rotation, and stay in registers.  Of 256 rows: 5.7 us a round, where the kernel above took 12.0 with all 120 pairs through LDS.
// Instances for 128 to 512 values, the blocks of ranks up to 256; larger blocks, of which none was timed, take the kernel above.
template <int CW>
__global__ __launch_bounds__(BJ_NT) void jacobi_short_round_kernel(double* __restrict__ H, int m, int round, double tol, double abs_floor, double small,
                                                                  unsigned long long* __restrict__ rotations)
{
    constexpr int L = BJ_NW * CW;
    __shared__ double Sw[BJ_NW][16][17];
    __shared__ double S[16][17], J[16][17];
    __shared__ int s_rotated;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int n = lane & 15, g = lane >> 4;
    int P, Q;
    block_pair(blockIdx.x, round, m / 8, P, Q);
    auto row_of = [&](int r) { return H + (size_t)(r < 8 ? 8 * P + r : 8 * Q + r - 8) * L + CW * wave; };
    double2 ga[CW / 8];                 // row n, columns 8 e + 2 g, + 1
    double xa[CW / 16][4];              // row 4 kk + g, column 16 u + n
    {
        const double* const row = row_of(n);
#pragma unroll
        for (int e = 0; e < CW / 8; ++e) ga[e] = *reinterpret_cast<const double2*>(row + 8 * e + 2 * g);
    }
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
        const double* const row = row_of(4 * kk + g);
#pragma unroll
        for (int u = 0; u < CW / 16; ++u) xa[u][kk] = row[16 * u + n];
    }
    d4 acc = {0, 0, 0, 0}, acc1 = {0, 0, 0, 0};
#pragma unroll
    for (int e = 0; e < CW / 8; ++e) {
        acc = mfma64(ga[e].x, ga[e].x, acc);
        acc1 = mfma64(ga[e].y, ga[e].y, acc1);
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) Sw[wave][4 * v + g][n] = acc[v] + acc1[v];
    __syncthreads();
    if (tid < 256) {
        const int r = tid >> 4, c = tid & 15;
        double t = 0;
#pragma unroll
        for (int w = 0; w < BJ_NW; ++w) t += Sw[w][r][c];
        S[r][c] = t;
    }
    __syncthreads();
    if (wave == 0) {
        const int turned = round == 0 ? rotate_all_pairs(S, J, lane, tol, abs_floor, small) : rotate_cross_pairs(S, J, lane, tol, abs_floor, small);
        if (lane == 0) s_rotated = turned;
    }
    __syncthreads();
    if (s_rotated == ORTHOGONAL) return;         // (uniform over the workgroup)
    if (tid == 0) count_rotation(rotations + blockIdx.x, s_rotated);
    double aJ[4];
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) aJ[kk] = J[4 * kk + g][n];
    d4 d[CW / 16];
#pragma unroll
    for (int u = 0; u < CW / 16; ++u) d[u] = d4{0, 0, 0, 0};
#pragma unroll
    for (int kk = 0; kk < 4; ++kk)
#pragma unroll
        for (int u = 0; u < CW / 16; ++u) d[u] = mfma64(aJ[kk], xa[u][kk], d[u]);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        double* const row = row_of(4 * v + g);
#pragma unroll
        for (int u = 0; u < CW / 16; ++u) row[16 * u + n] = d[u][v];
    }
}

// C[i][j] = beta * C[i][j] + alpha * sum_k A[i*ai + k*ak] * B[j*bj + k*bk], i < M, j < N, k < K (beta == 0: C is
// not read).  shape: GM_LOWER, only the tiles that touch the lower triangle (j0 <= i0) are computed (symmetric updates);
// GM_B_LOWER, B[j][k] is zero for k < j (a lower triangle): the contraction begins at the tile's first column; GM_A_LOWER, the same of
// A[i][k].  Workgroups go to the eight dies in turn, so the grid has the lower triangle's tiles and no others (a square grid with empty
// upper tiles gives the die of the first columns a quarter more than that of the last: 70 % of the compute units' time used), and tiles
// with the longest contractions come first.
// Bound by the fp64 matrix cores: 64 x 64 outputs per workgroup, a quarter per wavefront as 2 x 2 blocks of
// v_mfma_f64_16x16x4_f64 (64 cycles each), operands staged through LDS 32 k at a time and requested two stages ahead (16 k and one
// ahead: 256 x 4096 x 4096 took 277 us).  256 rows x 4096 are one workgroup per compute unit, so one wavefront per SIMD and
// nothing to do while it stages: in two parts, two workgroups a unit, 213 -> 174 us and 6 for the sum; with fragments of two k a
// lane (one 16-byte LDS read where two of 8 were) 168, 51 TFLOP/s.  The Gram matrix of 4096 x 8192: 2.8 ms (3.6 on the square grid).  Tiles of 128
// halve the operand traffic but leave fewer of them to share out (4.4 ms).  LDS rows of 34 doubles: the sixteen rows of a
// fragment start in different banks.
// part: null, or room for gridDim.z partial products, each over its share of k (gemm_sum_kernel adds them).
// C may be A or B where a workgroup reads all it needs of it before it writes (one tile of rows or columns): no __restrict__.
// a value at a uniform address and an offset of the lane's own, in bytes (a buffer load takes both as they are)
template <typename T>
__device__ __forceinline__ T load_at(const T* base, uint32_t off)
{
    const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(base), 0, -1, 0x00027000);
    if constexpr (sizeof(T) == 8) {
        typedef uint32_t u2 __attribute__((ext_vector_type(2)));
        return __builtin_bit_cast(T, (u2)__builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0));
    } else {
        return __builtin_bit_cast(T, (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0));
    }
}
enum { GM_FULL = 0, GM_LOWER = 1, GM_B_LOWER = 2, GM_A_LOWER = 3 };
constexpr int GM_TILE = 64, GM_KT = 32;

// Whether every byte that a lane reads of a stage of an operand lies within 32 bits of the tile's address there (with one of the strides
// 1, the other the length of a row: up to 2^32 / 63 / 4 = 17 million calibration tokens).  Beyond, gemm_kernel's FAR instance takes
// 64-bit indices throughout.
inline bool near_offsets(long row_stride, long k_stride, size_t size)
{
    return ((size_t)(GM_TILE - 1) * row_stride + (size_t)(GM_KT - 1) * k_stride + 1) * size <= 0xFFFFFFFFull;
}

// ADD: beta is not 0 and there are no parts; the tile of C is then requested before the contraction
struct alignas(16) GemmLds { double a[2][GM_TILE * (GM_KT + 2)], b[2][GM_TILE * (GM_KT + 2)]; };
template <typename TA, typename TB, bool FAR, bool ADD>
__device__ __forceinline__ void gemm_tile(const TA* A, long ai, long ak, const TB* B, long bj, long bk, double* C, long ldc, int M, int N, int K,
                                          double alpha, double beta, int shape, double* part, GemmLds& lds)
{
    constexpr int TILE = GM_TILE, KT = GM_KT, ST = KT + 2, E = TILE * KT / 256, FR = TILE / 32;
    auto& As = lds.a;
    auto& Bs = lds.b;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int n = lane & 15, g = lane >> 4;
    int ty = blockIdx.y, tx = blockIdx.x;
    if (shape == GM_LOWER) {                              // tile t of the lower triangle, row after row
        const int t = tx;
        ty = (int)((sqrtf(8.f * (float)t + 1.f) - 1.f) * 0.5f);
        ty = ty * (ty + 1) / 2 > t ? ty - 1 : ty;
        ty = (ty + 1) * (ty + 2) / 2 <= t ? ty + 1 : ty;
        tx = t - ty * (ty + 1) / 2;
    } else if (shape == GM_B_LOWER) {                     // columns, the longest contractions, first
        ty = blockIdx.x;
        tx = blockIdx.y;
    }
    const int i0 = ty * TILE, j0 = tx * TILE;
    const int wi = TILE / 2 * (wave & 1), wj = TILE / 2 * (wave >> 1);
    const int stages = (K - 1) / KT + 1, parts = gridDim.z, z = blockIdx.z;
    const int first = shape == GM_B_LOWER ? j0 / KT : shape == GM_A_LOWER ? i0 / KT : 0;
    const int sb = first + (int)((long)(stages - first) * z / parts), se = first + (int)((long)(stages - first) * (z + 1) / parts);
    // This thread's elements of a stage: consecutive threads along whichever index is contiguous in memory.  A lane's offsets
    // (32 bits, where near_offsets says that they fit) stay the same, the tile's address moves; rows beyond the last one re-read
    // it, never stored.
    int row_a[E], row_b[E];
    uint32_t off_a[E], off_b[E];
    const int k_a = ak == 1 ? tid % KT : tid / TILE, k_b = bk == 1 ? tid % KT : tid / TILE;
    const int dk_a = ak == 1 ? 0 : 256 / TILE, dk_b = bk == 1 ? 0 : 256 / TILE;
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int ra_ = ak == 1 ? tid / KT + 256 / KT * e : tid % TILE, rb_ = bk == 1 ? tid / KT + 256 / KT * e : tid % TILE;
        row_a[e] = i0 + ra_ < M ? ra_ : M - 1 - i0;
        row_b[e] = j0 + rb_ < N ? rb_ : N - 1 - j0;
        off_a[e] = (uint32_t)(row_a[e] * ai + (k_a + dk_a * e) * ak) * (uint32_t)sizeof(TA);
        off_b[e] = (uint32_t)(row_b[e] * bj + (k_b + dk_b * e) * bk) * (uint32_t)sizeof(TB);
    }
    const int la = ak == 1 ? tid / KT * ST + k_a : tid % TILE * ST + k_a, sa = ak == 1 ? 256 / KT * ST : 256 / TILE;
    const int lb = bk == 1 ? tid / KT * ST + k_b : tid % TILE * ST + k_b, sbk = bk == 1 ? 256 / KT * ST : 256 / TILE;
    const TA* const A0 = A + (size_t)i0 * ai;
    const TB* const B0 = B + (size_t)j0 * bj;
    TA ra[2][E];
    TB rb[2][E];
    auto fetch = [&](int set, int st) __attribute__((always_inline)) {
        const int k0 = st * KT;
        if (!FAR && K - k0 >= KT) {
#pragma unroll
            for (int e = 0; e < E; ++e) {
                ra[set][e] = load_at(A0 + (size_t)k0 * ak, off_a[e]);
                rb[set][e] = load_at(B0 + (size_t)k0 * bk, off_b[e]);
            }
        } else {
#pragma unroll
            for (int e = 0; e < E; ++e) {
                const int at_a = k_a + dk_a * e, at_b = k_b + dk_b * e, left = K - k0;      // (k0 + 31 may be beyond 31 bits)
                ra[set][e] = A0[(size_t)row_a[e] * ai + (size_t)(at_a < left ? k0 + at_a : K - 1) * ak];
                rb[set][e] = B0[(size_t)row_b[e] * bj + (size_t)(at_b < left ? k0 + at_b : K - 1) * bk];
                if (at_a >= left) ra[set][e] = 0;
                if (at_b >= left) rb[set][e] = 0;
            }
        }
    };
    auto stage = [&](int set, int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int e = 0; e < E; ++e) {
            As[buf][la + sa * e] = (double)ra[set][e];
            Bs[buf][lb + sbk * e] = (double)rb[set][e];
        }
    };
    d4 acc[FR][FR], old[FR][FR];
#pragma unroll
    for (int e = 0; e < FR; ++e)
#pragma unroll
        for (int f = 0; f < FR; ++f) acc[e][f] = d4{0, 0, 0, 0};
    auto contract = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int kp = 0; kp < KT / 8; ++kp) {             // (eight k a pair of MFMAs: lane group g has 2 g and 2 g + 1 of them, one 16-byte read)
            double2 a[FR], b[FR];
#pragma unroll
            for (int e = 0; e < FR; ++e) {
                a[e] = *reinterpret_cast<const double2*>(&As[buf][(wi + 16 * e + n) * ST + 8 * kp + 2 * g]);
                b[e] = *reinterpret_cast<const double2*>(&Bs[buf][(wj + 16 * e + n) * ST + 8 * kp + 2 * g]);
            }
#pragma unroll
            for (int e = 0; e < FR; ++e)
#pragma unroll
                for (int f = 0; f < FR; ++f) acc[e][f] = mfma64(a[e].x, b[f].x, acc[e][f]);
#pragma unroll
            for (int e = 0; e < FR; ++e)
#pragma unroll
                for (int f = 0; f < FR; ++f) acc[e][f] = mfma64(a[e].y, b[f].y, acc[e][f]);
        }
    };
    // Stage sb + i waits in LDS buffer i % 2 and, two stages ahead, in register set i % 2 (stages past the end: the last one, not
    // used).  No branch in the loop touches the accumulators: where paths meet the compiler copies them.
    if (sb < se) {
        fetch(0, sb);
        if constexpr (ADD) {                              // (an element outside C: the last one of its row or column, not used)
#pragma unroll
            for (int e = 0; e < FR; ++e)
#pragma unroll
                for (int f = 0; f < FR; ++f)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const int gi = i0 + wi + 16 * e + 4 * v + g, gj = j0 + wj + 16 * f + n;
                        old[e][f][v] = C[(size_t)(gi < M ? gi : M - 1) * ldc + (gj < N ? gj : N - 1)];
                    }
        }
        stage(0, 0);
        fetch(1, sb + 1 < se ? sb + 1 : se - 1);
        __syncthreads();
        int s = sb;
        for (; s + 1 < se; s += 2) {
            fetch(0, s + 2 < se ? s + 2 : se - 1);
            contract(0);
            stage(1, 1);
            __syncthreads();
            fetch(1, s + 3 < se ? s + 3 : se - 1);
            contract(1);
            stage(0, 0);
            __syncthreads();
        }
        if (s < se) contract(0);
    }
#pragma unroll
    for (int e = 0; e < FR; ++e)
#pragma unroll
        for (int f = 0; f < FR; ++f)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int gi = i0 + wi + 16 * e + 4 * v + g, gj = j0 + wj + 16 * f + n;
                if (gi < M && gj < N) {
                    if (part) {
                        part[((size_t)z * M + gi) * N + gj] = acc[e][f][v];
                    } else {
                        double c = alpha * acc[e][f][v];
                        if constexpr (ADD) c += beta * old[e][f][v];
                        C[(size_t)gi * ldc + gj] = c;
                    }
                }
            }
}

template <typename TA, typename TB, bool FAR, bool ADD>
__global__ __launch_bounds__(256, 2) void gemm_kernel(const TA* A, long ai, long ak, const TB* B, long bj, long bk, double* C, long ldc, int M, int N, int K,
                                                   double alpha, double beta, int shape, double* part)
{
    __shared__ GemmLds lds;
    gemm_tile<TA, TB, FAR, ADD>(A, ai, ak, B, bj, bk, C, ldc, M, N, K, alpha, beta, shape, part, lds);
}

// C = beta * C + alpha * (the partial products, in order); lower: where their tiles of 64 touch the lower triangle
__global__ __launch_bounds__(256) void gemm_sum_kernel(const double* __restrict__ part, int parts, double* __restrict__ C, long ldc, int M, int N, double alpha,
                                                       double beta, int lower)
{
    const size_t e = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= (size_t)M * N) return;
    const int i = (int)(e / N), j = (int)(e - (size_t)i * N);
    if (lower && j / 64 > i / 64) return;
    double v = 0.0;
    for (int z = 0; z < parts; ++z) v += part[(size_t)z * M * N + e];
    double c = alpha * v;
    if (beta != 0.0) c += beta * C[(size_t)i * ldc + j];
    C[(size_t)i * ldc + j] = c;
}

// the strict upper triangle of an n x n matrix from the lower one
__global__ __launch_bounds__(256) void mirror_kernel(double* __restrict__ A, int n)
{
    __shared__ double tile[32][33];
    const int bx = blockIdx.x * 32, by = blockIdx.y * 32, tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    if (bx > by) return;                      // source tile (by, bx) in or below the diagonal
    for (int e = ty; e < 32; e += 8)
        tile[e][tx] = (by + e < n && bx + tx < n) ? A[(size_t)(by + e) * n + bx + tx] : 0.0;
    __syncthreads();
    for (int e = ty; e < 32; e += 8)
        if (bx + e < n && by + tx < n && by + tx > bx + e) A[(size_t)(bx + e) * n + by + tx] = tile[tx][e];
}

// ------------------------------------------------------------------------------------------------------------
// Cholesky factor of the Gram matrix, G = L L^T, in place in the lower triangle (right-looking, blocks of 64):
// any S with S S^T = X~ X~^T serves Algorithm 1 as the eigenvectors times the roots of the eigenvalues do (the
// two differ by an orthogonal factor on the right, which the SVD of step 5 absorbs), and L costs n^3 / 3 flops.
constexpr int CH_NB = 64;

// thr[0] = rel * max_i G[i][i]: pivots at or below it make the factorisation give up (flag)
__global__ __launch_bounds__(1024) void pivot_floor_kernel(const double* __restrict__ G, int n, double rel, double* __restrict__ thr)
{
    __shared__ double red[1024];
    double m = 0.0;
    for (int i = threadIdx.x; i < n; i += 1024) m = fmax(m, G[(size_t)i * n + i]);
    red[threadIdx.x] = m;
    __syncthreads();
    for (int s2 = 512; s2 > 0; s2 >>= 1) {
        if ((int)threadIdx.x < s2) red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + s2]);
        __syncthreads();
    }
    if (threadIdx.x == 0) thr[0] = rel * red[0];
}

// The nb x nb diagonal block at (j0, j0), by one workgroup, as 4 x 4 blocks of 16 (rows beyond nb: those of the identity).  A
// block on the diagonal is factored in the registers of one wavefront, lane i % 16 its row i (right-looking, the column's entries passed by DPP), and inverted there, lane c column c; the blocks
// below and the trailing ones are products on the matrix cores.  The block's strict upper part is zeroed.  Then, unless
// inv is null, inv = L11^-1 (always 64 x 64, row-major), blockwise on the matrix cores too, so that the rows below the
// block and the right-hand sides of a solve are products.  Bound by the chain of 64 pivots.  (Left-looking over the whole 64
// columns by one wavefront, two LDS reads per multiplication: 94 us; with the inverse behind the factor 21; in one pass over the columns 19.)
// the value of lane LANE of the caller's row of 16 lanes
template <int LANE>
__device__ __forceinline__ double row_value(double v)
{
    const unsigned long long u = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = __builtin_amdgcn_mov_dpp((int)(unsigned)u, 0x150 + LANE, 0xF, 0xF, true);
    const unsigned hi = __builtin_amdgcn_mov_dpp((int)(unsigned)(u >> 32), 0x150 + LANE, 0xF, 0xF, true);
    return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}
template <int N, int I = 0, typename F>
__device__ __forceinline__ void unrolled(F&& f)
{
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        unrolled<N, I + 1>(f);
    }
}

// S: the matrix; once a column of blocks is done, the blocks of the inverse below the diagonal go to the mirrored places
// above it (block (i, j) of the inverse, i > j, at block (j, i), not transposed).  D: inverses of the diagonal blocks.
struct PotrfLds { double S[CH_NB][CH_NB + 2], D[4][16][18]; int bad; };
__device__ __forceinline__ void potrf_block(double* blk, long lda, int nb, const double* __restrict__ thr, unsigned* __restrict__ flag,
                                            double* __restrict__ inv, PotrfLds& lds)
{
    auto& S = lds.S;
    auto& D = lds.D;
    int& s_bad = lds.bad;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, n = lane & 15, g = lane >> 4;
    {
        double v[16];
        const int c = lane < nb ? lane : 0;
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const int r = wave + 4 * e;
            v[e] = blk[(size_t)(r < nb ? r : 0) * lda + c];
        }
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const int r = wave + 4 * e;
            S[r][lane] = r < nb && lane <= r ? v[e] : (lane == r ? 1.0 : 0.0);
        }
    }
    if (tid == 0) s_bad = 0;
    const double floor_abs = thr[0];
    __syncthreads();
#pragma unroll 1
    for (int jb = 0; jb < 4; ++jb) {
        if (wave == 0) {
            bool bad = false;
            double a[16], y[16];        // row n of the block; column n of its inverse (until y[j] is due: the identity's less what was eliminated)
#pragma unroll
            for (int c = 0; c < 16; ++c) {
                a[c] = S[16 * jb + n][16 * jb + c];
                y[c] = c == n ? 1.0 : 0.0;
            }
            double d, rinv;
            auto pivot = [&](auto jt) __attribute__((always_inline)) {
                constexpr int j = decltype(jt)::value;
                d = row_value<j>(a[j]);
                const bool low = 16 * jb + j < nb && !(d > floor_abs);       // not (numerically) positive definite: give up, stay finite
                bad = bad || low;
                d = low ? (floor_abs > 0.0 ? floor_abs : 1.0) : d;
                rinv = rsq_newton(d);
            };
            pivot(std::integral_constant<int, 0>{});
            unrolled<16>([&](auto jt) __attribute__((always_inline)) {
                constexpr int j = decltype(jt)::value;
                double root = d * rinv;
                root = fma(fma(-root, root, d), 0.5 * rinv, root);
                a[j] = n == j ? root : a[j] * rinv;
                y[j] *= rinv;
                // the next pivot's column first, so that its root is found beside the other columns' elimination
                unrolled<15 - j>([&](auto kt) __attribute__((always_inline)) {
                    constexpr int k = j + 1 + decltype(kt)::value;
                    const double l = row_value<k>(a[j]);  // (the entry that eliminates in the block and in its inverse)
                    a[k] = fma(-a[j], l, a[k]);
                    y[k] = fma(-l, y[j], y[k]);
                    if constexpr (k == j + 1) pivot(std::integral_constant<int, k>{});
                });
                // (or the compiler puts the elimination in the inverse off and keeps all 120 entries for it: 370 registers instead of 145)
#pragma unroll
                for (int c = 0; c < 16; ++c) asm volatile("" : "+v"(y[c]), "+v"(a[c]));
                __builtin_amdgcn_sched_barrier(0);
            });
            if (lane < 16) {
#pragma unroll
                for (int c = 0; c < 16; ++c) {
                    S[16 * jb + n][16 * jb + c] = c <= n ? a[c] : 0.0;
                    D[jb][c][n] = y[c];
                }
            }
            if (lane == 0 && bad) s_bad = 1;
        }
        __syncthreads();
        for (int ib = jb + 1 + wave; ib < 4; ib += 4) {   // block below: times L11^-T
            d4 x = {0, 0, 0, 0};
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) x = mfma64(S[16 * ib + n][16 * jb + 4 * kk + g], D[jb][n][4 * kk + g], x);
#pragma unroll
            for (int v = 0; v < 4; ++v) S[16 * ib + 4 * v + g][16 * jb + n] = x[v];
        }
        __syncthreads();
        int turn = 0;
#pragma unroll 1
        for (int ib = jb + 1; ib < 4; ++ib)
#pragma unroll 1
            for (int kb = jb + 1; kb <= ib; ++kb) {
                if ((turn++ & 3) != wave) continue;
                d4 c;
#pragma unroll
                for (int v = 0; v < 4; ++v) c[v] = S[16 * ib + 4 * v + g][16 * kb + n];
#pragma unroll
                for (int kk = 0; kk < 4; ++kk) c = mfma64(-S[16 * ib + n][16 * jb + 4 * kk + g], S[16 * kb + n][16 * jb + 4 * kk + g], c);
#pragma unroll
                for (int v = 0; v < 4; ++v) S[16 * ib + 4 * v + g][16 * kb + n] = c[v];
            }
        __syncthreads();
    }
    if (tid == 0 && s_bad) atomicOr(flag, 1u);
#pragma unroll
    for (int e = 0; e < 16; ++e) {
        const int r = wave + 4 * e;
        if (r < nb && lane < nb) blk[(size_t)r * lda + lane] = lane <= r ? S[r][lane] : 0.0;
    }
    if (!inv) return;
    // X(i, j) = -D(i) sum over j <= k < i of L(i, k) X(k, j): the three diagonals of blocks below the main one in turn, a block a
    // wavefront (the places above the diagonal they go to are zeros that nobody reads as L any more)
    __syncthreads();
#pragma unroll 1
    for (int dist = 1; dist < 4; ++dist) {
        const int j = wave, i = wave + dist;
        if (i < 4) {
            d4 w = {0, 0, 0, 0}, x = {0, 0, 0, 0};
#pragma unroll 1
            for (int k = j; k < i; ++k)
#pragma unroll
                for (int kk = 0; kk < 4; ++kk)
                    w = mfma64(S[16 * i + n][16 * k + 4 * kk + g], k == j ? D[j][4 * kk + g][n] : S[16 * j + 4 * kk + g][16 * k + n], w);
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) x = mfma64(D[i][n][4 * kk + g], w[kk], x);      // (register kk of w is row 4 kk + g: the operand)
#pragma unroll
            for (int v = 0; v < 4; ++v) S[16 * j + 4 * v + g][16 * i + n] = -x[v];
        }
        __syncthreads();
    }
#pragma unroll
    for (int e = 0; e < 16; ++e) {
        const int r = wave + 4 * e, bi = r >> 4, bj = lane >> 4;
        const double below = S[16 * bj + (r & 15)][16 * bi + n], diag = D[bi][r & 15][n];
        inv[r * CH_NB + lane] = bi < bj ? 0.0 : bi == bj ? diag : below;
    }
}

// the first diagonal block, nb x nb at A
__global__ __launch_bounds__(256, 2) void potrf_block_kernel(double* A, long lda, int nb, const double* __restrict__ thr, unsigned* __restrict__ flag, double* __restrict__ inv)
{
    __shared__ PotrfLds lds;
    potrf_block(A, lda, nb, thr, flag, inv, lds);
}

// The trailing matrix C (rest x rest) less P P^T (P: rest x nb), and its first block, the next diagonal one, factored by the
// workgroup that has just finished it: the chain of diagonal blocks (20 us each, one workgroup) goes on beside the other
// tiles (8 to 70 us).  4096 x 4096, rank 128: 32.0 -> 31.3 ms.
__global__ __launch_bounds__(256, 2) void update_factor_kernel(const double* P, double* C, long ld, int rest, int nb, const double* __restrict__ thr,
                                                              unsigned* __restrict__ flag, double* __restrict__ inv)
{
    __shared__ union { GemmLds g; PotrfLds p; } lds;
    gemm_tile<double, double, false, true>(P, ld, 1L, P, ld, 1L, C, ld, rest, rest, nb, -1.0, 1.0, GM_LOWER, nullptr, lds.g);
    if (blockIdx.x != 0) return;
    __syncthreads();                                      // the tile is in memory, its operands in LDS are dead
    potrf_block(C, ld, rest < CH_NB ? rest : CH_NB, thr, flag, inv, lds.p);
}

__global__ void zero_upper_kernel(double* __restrict__ A, int n)
{
    const size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= (size_t)n * n) return;
    const int i = (int)(e / n), c = (int)(e - (size_t)i * n);
    if (c > i) A[e] = 0.0;
}

// dst[c][i] = src[i][c] for an n x n matrix
__global__ void transpose_kernel(const double* __restrict__ src, double* __restrict__ dst, int n)
{
    __shared__ double tile[32][33];
    const int bx = blockIdx.x * 32, by = blockIdx.y * 32, tx = threadIdx.x & 31, ty = threadIdx.x >> 5;      // 256 threads: 32 x 8
    for (int e = ty; e < 32; e += 8)
        tile[e][tx] = (by + e < n && bx + tx < n) ? src[(size_t)(by + e) * n + bx + tx] : 0.0;
    __syncthreads();
    for (int e = ty; e < 32; e += 8)
        if (bx + e < n && by + tx < n) dst[(size_t)(bx + e) * n + by + tx] = tile[tx][e];
}

__global__ void iota_kernel(int* __restrict__ idx, int r)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < r) idx[i] = i;
}

// Bn[i][o] = B[o][i] / sigma[i]^2 (B: d_out x r)
__global__ void scaled_transpose_kernel(const double* __restrict__ B, const double* __restrict__ sigma, int d_out, int r,
                                        double* __restrict__ Bn)
{
    const size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= (size_t)d_out * r) return;
    const int i = (int)(e / d_out), o = (int)(e - (size_t)i * d_out);
    const double sg = sigma[i];
    Bn[e] = sg > 0.0 ? B[(size_t)o * r + i] / (sg * sg) : 0.0;
}

__global__ void sub_kernel(const float* __restrict__ W, const float* __restrict__ What, double* __restrict__ dW, size_t n)
{
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dW[i] = (double)W[i] - (double)What[i];
}

__global__ void identity_kernel(double* __restrict__ V, int m)
{
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < (size_t)m * m) V[i] = (i / m == i % m) ? 1.0 : 0.0;
}

__global__ void copy_kernel(const double* __restrict__ src, double* __restrict__ dst, size_t n)
{
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dst[i] = src[i];
}

__global__ void clear_flag_kernel(unsigned* flag) { *flag = 0; }

__global__ void clear_counters_kernel(unsigned long long* __restrict__ c, int n)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) c[i] = 0;
}

// out[p] = sum_k X[p][k] * Y[p][k]; one workgroup of 256 per row
__global__ __launch_bounds__(256) void row_dot_kernel(const double* __restrict__ X, const double* __restrict__ Y, int L,
                                                      double* __restrict__ out)
{
    const int p = blockIdx.x;
    double s = 0;
    for (int k = threadIdx.x; k < L; k += 256) s += X[(size_t)p * L + k] * Y[(size_t)p * L + k];
    __shared__ double red[4];
    s = wave_sum(s);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) out[p] = red[0] + red[1] + red[2] + red[3];
}

// root[p] = sqrt(max(lam[p], floor * max lam)), inv[p] = 1 / root[p]; one workgroup
__global__ __launch_bounds__(1024) void eig_roots_kernel(const double* __restrict__ lam, int m, double floor_rel,
                                                         double* __restrict__ root, double* __restrict__ inv)
{
    __shared__ double red[16];
    __shared__ double top;
    double mx = -INFINITY;
    for (int k = threadIdx.x; k < m; k += 1024) mx = fmax(mx, lam[k]);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) mx = fmax(mx, __shfl_xor(mx, o, 64));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = mx;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = red[0];
        for (int w = 1; w < 16; ++w) t = fmax(t, red[w]);
        top = t;
    }
    __syncthreads();
    for (int k = threadIdx.x; k < m; k += 1024) {
        const double r = sqrt(fmax(lam[k], floor_rel * top));
        root[k] = r;
        inv[k] = 1.0 / r;
    }
}

// X[p][k] *= (by_row ? s[p] : s[k])
__global__ void scale_kernel(double* __restrict__ X, int rows, int L, const double* __restrict__ s, int by_row)
{
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < (size_t)rows * L) X[i] *= by_row ? s[i / L] : s[i % L];
}

// idx[rank] = p for the r rows of largest sq (ties: lower row first); sigma[rank] = sqrt(sq[p])
__global__ void top_rows_kernel(const double* __restrict__ sq, int m, int r, int* __restrict__ idx, double* __restrict__ sigma)
{
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= m) return;
    const double v = sq[p];
    int rank = 0;
    for (int q = 0; q < m; ++q) {
        const double u = sq[q];
        rank += (u > v) || (u == v && q < p);
    }
    if (rank < r) {
        idx[rank] = p;
        sigma[rank] = sqrt(v);
    }
}

// dst[i][k] = src[idx[i]][k] * sigma[i]^power   (power = -1: unit rows; 0: copy; -2: divided by the square)
__global__ void gather_rows_kernel(const double* __restrict__ src, int L, const int* __restrict__ idx,
                                   const double* __restrict__ sigma, int power, double* __restrict__ dst, int r)
{
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (size_t)r * L) return;
    const int row = (int)(i / L), k = (int)(i % L);
    const double s = sigma[row];
    // a vanishing singular value (error of rank below r, or no error at all) gives a zero component, not 0/0
    const double f = power == 0 ? 1.0 : (s > 0.0 ? (power == -1 ? 1.0 / s : 1.0 / (s * s)) : 0.0);
    dst[i] = src[(size_t)idx[row] * L + k] * f;
}

// dst[o][i] = src[idx[i]][o]   (dst: L x r)
__global__ void gather_rows_transposed_kernel(const double* __restrict__ src, int L, const int* __restrict__ idx,
                                              double* __restrict__ dst, int r)
{
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (size_t)r * L) return;
    const int o = (int)(i / r), c = (int)(i % r);
    dst[i] = src[(size_t)idx[c] * L + o];
}

// s[i] = sqrt(|B'_i| / |A_i|) for component i (column i of B: d_out x r, row i of A: r x d_in), 1 if either
// vanishes; one workgroup of 256 per component
__global__ __launch_bounds__(256) void balance_kernel(const double* __restrict__ B, const double* __restrict__ A, int d_in,
                                                      int d_out, int r, double* __restrict__ s)
{
    const int i = blockIdx.x;
    double nb = 0, na = 0;
    for (int o = threadIdx.x; o < d_out; o += 256) nb += B[(size_t)o * r + i] * B[(size_t)o * r + i];
    for (int k = threadIdx.x; k < d_in; k += 256) na += A[(size_t)i * d_in + k] * A[(size_t)i * d_in + k];
    __shared__ double red[2][4];
    nb = wave_sum(nb);
    na = wave_sum(na);
    if ((threadIdx.x & 63) == 0) {
        red[0][threadIdx.x >> 6] = nb;
        red[1][threadIdx.x >> 6] = na;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        nb = sqrt(red[0][0] + red[0][1] + red[0][2] + red[0][3]);
        na = sqrt(red[1][0] + red[1][1] + red[1][2] + red[1][3]);
        s[i] = (nb > 0.0 && na > 0.0) ? sqrt(nb / na) : 1.0;
    }
}

// One thread per (tile, lane) of the F16 tile layout (tile = 16 rows x 32 columns, lane l = 16 j + n owns row n,
// columns 8 j .. 8 j + 7): eight values of X (rows x K fp64 row-major), scaled, rounded once to fp16.
// by_row: the scale of a value is s[row] (A: times s) or 1 / s[column] (B: divided by s); s == nullptr: 1.
__global__ void store_f16_tiles_kernel(const double* __restrict__ X, int rows, int K, const double* __restrict__ s, int by_row,
                                       _Float16* __restrict__ out)
{
    const size_t L = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (L >= (size_t)rows * K / 8) return;
    const int ntk = K / 32;
    const size_t tile = L / 64;
    const int lane = (int)(L % 64);
    const int R = (int)(tile / ntk), g = (int)(tile % ntk);
    const int j = lane >> 4, n = lane & 15;
    const int row = 16 * R + n, col0 = 32 * g + 8 * j;
    for (int i = 0; i < 8; ++i) {
        double v = X[(size_t)row * K + col0 + i];
        if (s) v = by_row ? v * s[row] : v / s[col0 + i];
        out[L * 8 + i] = (_Float16)v;
    }
}

// Symmetric quantisation of a factor X (rows x K fp64) into the Q4 (BITS = 4, KT = 128 or 64) or Q3 (BITS = 3,
// KT = 128) tile layout with one fp16 scale per row and group of KT columns (Sec. 4.5, App. A.9: quantised
// factors).  One wavefront per tile: lane l = 16 j + n owns row n and columns (KT/4) j .. of the tile; the four
// lanes of a row find the group's largest magnitude with two shuffles.  scale = fp16(max |v| / qpos)
// (1 for an all-zero group), code = clip(rint(v / scale) + zp, 1, 2 zp - 1), zp = 2^(BITS-1), qpos = zp - 1.
// s / by_row: the balancing scale of store_f16_tiles_kernel.
template <int BITS, int KT>
__global__ __launch_bounds__(64) void store_q_tiles_kernel(const double* __restrict__ X, int rows, int K, const double* __restrict__ s,
                                                           int by_row, uint32_t* __restrict__ out, _Float16* __restrict__ scales)
{
    constexpr int CPL = KT / 4, ZP = 1 << (BITS - 1), QPOS = ZP - 1;
    const int tile = blockIdx.x, lane = threadIdx.x;
    const int ntk = K / KT;
    const int R = tile / ntk, g = tile % ntk;
    const int j = lane >> 4, n = lane & 15;
    const int row = 16 * R + n, col0 = KT * g + CPL * j;
    double v[CPL];
    double amax = 0.0;
#pragma unroll
    for (int c = 0; c < CPL; ++c) {
        double x = X[(size_t)row * K + col0 + c];
        if (s) x = by_row ? x * s[row] : x / s[col0 + c];
        v[c] = x;
        amax = fmax(amax, fabs(x));
    }
    amax = fmax(amax, __shfl_xor(amax, 16, 64));
    amax = fmax(amax, __shfl_xor(amax, 32, 64));
    _Float16 sc = (_Float16)(amax / (double)QPOS);
    if (sc == (_Float16)0.0f) sc = (_Float16)1.0f;
    const double scd = (double)sc;
    uint32_t code[CPL];
#pragma unroll
    for (int c = 0; c < CPL; ++c) {
        double q = rint(v[c] / scd) + (double)ZP;
        q = fmin(fmax(q, 1.0), (double)(2 * ZP - 1));
        code[c] = (uint32_t)q;
    }
    if (j == 0) scales[(size_t)row * ntk + g] = sc;
    if constexpr (BITS == 4) {
        constexpr int WPL = KT / 32;
#pragma unroll
        for (int t = 0; t < WPL; ++t) {
            uint32_t w = 0;
#pragma unroll
            for (int kk = 0; kk < 8; ++kk) w |= code[8 * t + kk] << (4 * (4 * (kk % 2) + kk / 2));
            out[((size_t)tile * 64 + lane) * WPL + t] = w;
        }
    } else {
        uint32_t d[3] = {0u, 0u, 0u};
#pragma unroll
        for (int cc = 0; cc < 30; ++cc) d[(cc / 2) / 5] |= code[cc] << (16 * (cc % 2) + 3 * ((cc / 2) % 5));
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int b = 0; b < 3; ++b) d[b] |= ((code[30 + h] >> b) & 1u) << (16 * h + 15);
#pragma unroll
        for (int b = 0; b < 3; ++b) out[((size_t)tile * 64 + lane) * 3 + b] = d[b];
    }
}

// ------------------------------------------------------------------------------------------------------------
// The r leading left singular vectors of T (m x n) by Chebyshev-filtered subspace iteration on S = T T^T, for r well
// below m: the Jacobi sweeps over all m rows compute m components of which r are kept.  A block of p >= 2 r vectors
// (rows of Z, length m) is filtered with a Chebyshev polynomial that is bounded by 1 on [0, a], a = the smallest Ritz
// value of the block, orthonormalised (Cholesky of its Gram matrix, twice) and rotated to its Ritz vectors; the degree
// is what the spread of the Ritz values allows before the smallest directions drown in the rounding of the largest.
// Leading vectors that have converged are taken out once that lowers the spread.  Convergence needs the gap to the
// (p + 1)-th singular value only; the r-th is told from the (r + 1)-th by the Jacobi sweeps over the p rows of Z T at the
// end.  (Zhou, Saad, Tiago, Chelikowsky 2006.)
//  - A locked vector keeps an error of SUB_TOL of its own Ritz value, which couples it to the others.  That coupling stays
//    inside the block and the sweeps at the end undo it, so it is no residual of theirs: Y = Z S is taken orthogonal to the
//    locked rows.  (Counted, it held inputs whose outlier channels are 60 times the rest or more above SUB_TOL for good.)
//  - S has the rounding of sigma_1^2 in every entry: a direction of sigma_r is off by about 1e-16 (sigma_1 / sigma_r)^2.
//    As long as the spread of the Ritz values is at most SUB_DOWNDATE the locked vectors are taken out of S itself (that
//    error is then below SUB_TOL); beyond, out of T, and S is formed again (T - X^T (X T) has the rounding of sigma_1 only).
//    Largest angle between the r leading vectors and the block, numpy model, 1024 rows, r = 32 and 100, outliers 60 to 3000
//    times the rest: 2e-12, at a spread sigma_1 / sigma_r of 3110.

// deterministic entries in (-1, 1)
__global__ void random_rows_kernel(double* __restrict__ Z, size_t n)
{
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    unsigned long long x = (i + 1) * 0x9E3779B97F4A7C15ull;      // splitmix64 (Steele, Lea, Flood 2014)
    x = (x ^ (x >> 30)) * 0xBF58476D1CE4E5B9ull;
    x = (x ^ (x >> 27)) * 0x94D049BB133111EBull;
    x ^= x >> 31;
    Z[i] = (double)(long long)x * (1.0 / 9223372036854775808.0);
}

__global__ void add_diagonal_kernel(double* __restrict__ S, int m, double v)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < m) S[(size_t)i * m + i] += v;
}

// row p of Z divided by its norm; one workgroup of 256 per row
__global__ __launch_bounds__(256) void normalise_rows_kernel(double* __restrict__ Z, int L)
{
    double* const z = Z + (size_t)blockIdx.x * L;
    double s = 0;
    for (int k = threadIdx.x; k < L; k += 256) s += z[k] * z[k];
    __shared__ double red[4];
    s = wave_sum(s);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    s = red[0] + red[1] + red[2] + red[3];
    const double f = s > 0.0 ? 1.0 / sqrt(s) : 0.0;
    for (int k = threadIdx.x; k < L; k += 256) z[k] *= f;
}

// out[p] = | Y_p - theta[p] Z_p |, one workgroup of 256 per row
__global__ __launch_bounds__(256) void residual_kernel(const double* __restrict__ Y, const double* __restrict__ Z, int L,
                                                       const double* __restrict__ theta, double shift, double* __restrict__ out)
{
    const int p = blockIdx.x;
    const double t = theta[p] - shift;
    double s = 0;
    for (int k = threadIdx.x; k < L; k += 256) {
        const double d = Y[(size_t)p * L + k] - t * Z[(size_t)p * L + k];
        s += d * d;
    }
    __shared__ double red[4];
    s = wave_sum(s);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) out[p] = sqrt(red[0] + red[1] + red[2] + red[3]);
}

// G (p x p): the first nl rows and columns become diag(theta), `shift` is added to the rest of the diagonal, and the
// rest is made symmetric
__global__ void ritz_matrix_kernel(const double* __restrict__ src, double* __restrict__ G, int p, int nl, const double* __restrict__ theta, double shift)
{
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= p * p) return;
    const int i = e / p, c = e - i * p;
    double v;
    if (i < nl || c < nl) v = i == c ? theta[i] : 0.0;
    else v = 0.5 * (src[(size_t)i * p + c] + src[(size_t)c * p + i]) + (i == c ? shift : 0.0);
    G[e] = v;
}

// rank of lam[i], the squared norm of row i of R, among p values (descending): out row rank <- that row divided by its norm, theta[rank] = lam[i]
__global__ __launch_bounds__(256) void sort_rows_kernel(const double* __restrict__ R, const double* __restrict__ lam, int p, double* __restrict__ out,
                                                        double* __restrict__ theta)
{
    __shared__ int s_rank;
    const int i = blockIdx.x;
    if (threadIdx.x == 0) s_rank = 0;
    __syncthreads();
    const double v = lam[i];
    int rank = 0;
    for (int q = threadIdx.x; q < p; q += 256) rank += (lam[q] > v) || (lam[q] == v && q < i);
    atomicAdd(&s_rank, rank);
    __syncthreads();
    rank = s_rank;
    if (threadIdx.x == 0) theta[rank] = v;
    const double f = v > 0.0 ? 1.0 / sqrt(v) : 0.0;
    for (int k = threadIdx.x; k < p; k += 256) out[(size_t)rank * p + k] = R[(size_t)i * p + k] * f;
}

inline unsigned blocks(size_t n, int per = 256) { return (unsigned)((n + per - 1) / per); }

// (a launch like the others: its error is the call's, where an unchecked copy's would be lost)
void copy_doubles(const double* src, double* dst, size_t n, hipStream_t st)
{
    hipLaunchKernelGGL(copy_kernel, dim3(blocks(n)), dim3(256), 0, st, src, dst, n);
}

// Parts of the contraction of a product of `tiles` tiles whose caller has `room` doubles of scratch: where there are few tiles and a long
// contraction the compute units share it (256 x 256 with k = 4096: 10 tiles take 260 us, in parts 18, and 5 for their sum); the parts are
// added in order.  From 65 to 511 tiles the parts that cost least of those that have at least four stages each and fit the scratch: a column of the contraction
// takes 0.08 us with two workgroups a unit and 0.052 with one, full rounds of 512 come first and what is left over after them; then the partial
// sums written and read.  Whole calls, in ms, with one to five parts of each product with S: 3072 x 3072, rank 192 (288 tiles) 30.1, 28.4, 27.7, 27.6, 27.5;
// 2304 x 2304, rank 128 (144) 17.5, 16.8, 16.0, 16.2, 15.9; 5120 x 5120, rank 128 (320) 48.9, 44.1, 42.7, 42.2, 43.3; 2560 x 2560, rank 224 (320) 33.5, 32.5
// and no room for more; 3072 x 3072, rank 256 (384) 36.9, 35.7, 36.2.  (With every begun round at 0.08 the cost says one part for the last two.)
int gemm_parts(int tiles, int M, int N, int K, size_t room)
{
    if (tiles >= 512 || K < 512) return 1;
    size_t most = room / ((size_t)M * N);
    if (most > (size_t)K / 128) most = K / 128;
    if (tiles <= 64) return (int)(most < 1 ? 1 : most < (size_t)(256 / tiles) ? most : 256 / tiles);
    float best = 1e30f;
    int parts = 1;
    for (int c = 1; c <= 8 && (c == 1 || (size_t)c <= most); ++c) {
        const int left = tiles * c % 512;
        const float column = 0.08f * (float)(tiles * c / 512) + (left == 0 ? 0.f : left <= 256 ? 0.052f : 0.08f);
        const float us = column * (float)K / (float)c + (c > 1 ? 4.f + 4e-6f * (float)M * (float)N * (float)c : 0.f);
        if (us < best) {
            best = us;
            parts = c;
        }
    }
    return parts;
}

template <typename TA, typename TB>
void gemm(const TA* A, long ai, long ak, const TB* B, long bj, long bk, double* C, long ldc, int M, int N, int K,
          hipStream_t st, double alpha = 1.0, double beta = 0.0, int shape = GM_FULL, double* scratch = nullptr, size_t room = 0)
{
    const int ti = (M + 63) / 64, tj = (N + 63) / 64, tiles = shape == GM_LOWER ? ti * (ti + 1) / 2 : ti * tj;
    dim3 grid = shape == GM_LOWER ? dim3(tiles) : shape == GM_B_LOWER ? dim3(ti, tj) : dim3(tj, ti);
    auto kern = gemm_kernel<TA, TB, false, false>;
    // (fp64 operands are matrices of at most MAX_DIM columns.  An instance of its own: tested in the kernel instead, a call at
    // 4096 x 4096 takes 46.5 ms instead of 46.1)
    if constexpr (std::is_same_v<TA, float>)
        if (!near_offsets(ai, ak, sizeof(TA)) || !near_offsets(bj, bk, sizeof(TB))) kern = gemm_kernel<TA, TB, true, false>;            // (no call with calibration tokens adds to C)
    if (scratch && (shape == GM_FULL || shape == GM_LOWER)) {
        const int parts = gemm_parts(tiles, M, N, K, room);
        if (parts > 1) {
            grid.z = (unsigned)parts;
            hipLaunchKernelGGL(kern, grid, dim3(256), 0, st, A, ai, ak, B, bj, bk, C, ldc, M, N, K, alpha, beta, shape, scratch);
            hipLaunchKernelGGL(gemm_sum_kernel, dim3(blocks((size_t)M * N)), dim3(256), 0, st, (const double*)scratch, parts, C, ldc, M, N, alpha, beta,
                               shape == GM_LOWER);
            return;
        }
    }
    if constexpr (std::is_same_v<TA, double>)
        if (beta != 0.0) kern = gemm_kernel<TA, TB, false, true>;
    hipLaunchKernelGGL(kern, grid, dim3(256), 0, st, A, ai, ak, B, bj, bk, C, ldc, M, N, K, alpha, beta, shape, (double*)nullptr);
}
static_assert(((size_t)(GM_TILE - 1) * MAX_DIM + GM_KT) * sizeof(double) <= 0xFFFFFFFFull, "fp64 operands have near offsets");

// G (n x n, row-major, symmetric) -> L in its lower triangle, zeros above.  Enqueues only; *flag (device, cleared
// here) is raised if a pivot is not above rel * max diag(G): the factor is then unusable.
// clear == false leaves a flag that is already up.  inv: scratch of CH_NB^2 doubles, not touched when n <= CH_NB (a
// matrix of one block has no rows below it; a scratch of n x n is then smaller than an inverse); or, keep_inv, one such
// block per diagonal block, which then holds their inverses.
void cholesky(double* G, int n, double rel, double* thr, unsigned* flag, double* inv, hipStream_t st, bool clear = true, bool keep_inv = false)
{
    if (clear) hipLaunchKernelGGL(clear_flag_kernel, dim3(1), dim3(1), 0, st, flag);
    hipLaunchKernelGGL(pivot_floor_kernel, dim3(1), dim3(1024), 0, st, G, n, rel, thr);
    for (int j0 = 0; j0 < n; j0 += CH_NB) {
        const int nb = n - j0 < CH_NB ? n - j0 : CH_NB, rest = n - j0 - nb;
        double* const iv = inv + (keep_inv ? (size_t)j0 * CH_NB : 0);
        if (j0 == 0) hipLaunchKernelGGL(potrf_block_kernel, dim3(1), dim3(256), 0, st, G, (long)n, nb, thr, flag, keep_inv || rest > 0 ? iv : nullptr);
        if (rest <= 0) break;
        // rows below: P <- P L11^-T, in place (a workgroup reads its 64 rows whole before it writes them)
        double* const P = G + (size_t)(j0 + nb) * n + j0;
        gemm((const double*)P, (long)n, 1L, (const double*)iv, (long)CH_NB, 1L, P, (long)n, rest, nb, nb, st);
        // trailing matrix -= panel . panel^T (the tiles of its lower triangle), and the next diagonal block (whose inverse may take this one's place)
        const int ti = (rest + GM_TILE - 1) / GM_TILE;
        hipLaunchKernelGGL(update_factor_kernel, dim3(ti * (ti + 1) / 2), dim3(256), 0, st, (const double*)P, G + (size_t)(j0 + nb) * n + (j0 + nb), (long)n, rest, nb,
                           (const double*)thr, flag, keep_inv ? iv + (size_t)nb * CH_NB : rest > CH_NB ? iv : nullptr);
    }
    hipLaunchKernelGGL(zero_upper_kernel, dim3(blocks((size_t)n * n)), dim3(256), 0, st, G, n);
}

bool block_rounds_fit(int L, bool with_v, int m) { return m % 16 == 0 && m >= 32 && L % 128 == 0 && (!with_v || m % 128 == 0); }

void jacobi_round(double* H, int L, double* V, int m, int round, double tol, double abs_floor, double small, unsigned long long* counters, hipStream_t st)
{
    const dim3 g(m / 2);
    const int need = (L / 2 + JPT - 1) / JPT;          // threads that cover a row
    if (need <= 64)
        hipLaunchKernelGGL(jacobi_round_kernel<64>, g, dim3(64), 0, st, H, L, V, m, round, tol, abs_floor, small, counters);
    else if (need <= 128)
        hipLaunchKernelGGL(jacobi_round_kernel<128>, g, dim3(128), 0, st, H, L, V, m, round, tol, abs_floor, small, counters);
    else if (need <= 256)
        hipLaunchKernelGGL(jacobi_round_kernel<256>, g, dim3(256), 0, st, H, L, V, m, round, tol, abs_floor, small, counters);
    else if (need <= 512)
        hipLaunchKernelGGL(jacobi_round_kernel<512>, g, dim3(512), 0, st, H, L, V, m, round, tol, abs_floor, small, counters);
    else
        hipLaunchKernelGGL(jacobi_round_kernel<1024>, g, dim3(1024), 0, st, H, L, V, m, round, tol, abs_floor, small, counters);
}

// Sweeps until one passes without a rotation that is not small (rotation_large).  Synchronises the stream once per sweep.  sq: m doubles of
// scratch.  Returns the number of sweeps, or -1 if MAX_SWEEPS did not suffice, or -2 on a runtime error.
// stats (may be null): sweeps, milliseconds between two events around the sweeps, workgroups that rotated
// their rows, rows per workgroup (2: pair rounds, 16: block rounds).
int jacobi_sweeps(double* H, int L, double* V, int m, double* sq, hipStream_t st, double* rotations);

int jacobi(double* H, int L, double* V, int m, double* sq, hipStream_t st, double* stats)
{
    hipEvent_t e0 = nullptr, e1 = nullptr;
    const bool timed = stats && hipEventCreate(&e0) == hipSuccess && hipEventCreate(&e1) == hipSuccess;
    if (timed) hipEventRecord(e0, st);
    double rotations = 0;
    const int sweeps = jacobi_sweeps(H, L, V, m, sq, st, &rotations);
    if (timed) {
        float ms = 0;
        hipEventRecord(e1, st);
        hipEventSynchronize(e1);
        hipEventElapsedTime(&ms, e0, e1);
        stats[0] = sweeps;
        stats[1] = ms;
        stats[2] = rotations;
        stats[3] = (block_rounds_fit(L, V != nullptr, m)) ? 16 : 2;
    }
    if (e0) hipEventDestroy(e0);
    if (e1) hipEventDestroy(e1);
    return sweeps;
}

int jacobi_sweeps(double* H, int L, double* V, int m, double* sq, hipStream_t st, double* rotations)
{
    // rows far below the largest are zero for every purpose here, and rotating them would never settle
    hipLaunchKernelGGL(row_dot_kernel, dim3(m), dim3(256), 0, st, H, H, L, sq);
    double* host = (double*)malloc(sizeof(double) * m);
    if (!host) return -2;
    if (hipMemcpyAsync(host, sq, sizeof(double) * m, hipMemcpyDeviceToHost, st) != hipSuccess ||
        hipStreamSynchronize(st) != hipSuccess) {
        free(host);
        return -2;
    }
    double top = 0;
    for (int p = 0; p < m; ++p) top = host[p] > top ? host[p] : top;
    const double abs_floor = top * 1e-30;
    const double tol = sqrt((double)L) * 1.1102230246251565e-16, small = sqrt(tol / (4.0 * m));
    // the counters of a round's workgroups (count_rotation) in place of the norms, cleared once and read after each sweep
    const bool by_blocks = block_rounds_fit(L, V != nullptr, m);
    const int workgroups = by_blocks ? m / 16 : m / 2;
    unsigned long long* const counters = reinterpret_cast<unsigned long long*>(sq);
    unsigned long long* const counted = reinterpret_cast<unsigned long long*>(host);
    hipLaunchKernelGGL(clear_counters_kernel, dim3(blocks(workgroups)), dim3(256), 0, st, counters, workgroups);
    unsigned long long large = 0;
    int result = -1;
    *rotations = 0;
    for (int sweep = 1; sweep <= MAX_SWEEPS && result == -1; ++sweep) {
        if (by_blocks) {
            auto short_rows = V ? nullptr : L == 128 ? jacobi_short_round_kernel<16> : L == 256 ? jacobi_short_round_kernel<32> :
                              L == 384 ? jacobi_short_round_kernel<48> : L == 512 ? jacobi_short_round_kernel<64> : nullptr;
            for (int round = 0; round < m / 8 - 1; ++round) {
                if (short_rows) hipLaunchKernelGGL(short_rows, dim3(workgroups), dim3(BJ_NT), 0, st, H, m, round, tol, abs_floor, small, counters);
                else hipLaunchKernelGGL(jacobi_block_round_kernel, dim3(workgroups), dim3(BJ_NT), 0, st, H, L, V, m, round, tol, abs_floor, small, counters);
            }
        } else {
            for (int round = 0; round < m - 1; ++round) jacobi_round(H, L, V, m, round, tol, abs_floor, small, counters, st);
        }
        if (hipMemcpyAsync(counted, counters, sizeof(*counted) * workgroups, hipMemcpyDeviceToHost, st) != hipSuccess ||
            hipStreamSynchronize(st) != hipSuccess) {
            result = -2;
            break;
        }
        unsigned long long all = 0, not_small = 0;         // rounds of workgroups that rotated rows, those of them with a rotation that was not small
        for (int i = 0; i < workgroups; ++i) {
            all += counted[i] & 0xFFFFFFFFull;
            not_small += counted[i] >> 32;
        }
        if (getenv("EORA_VERBOSE"))
            fprintf(stderr, "eora: jacobi m=%d L=%d sweep %d: %.0f rotations, %llu large\n", m, L, sweep, (double)all - *rotations, not_small - large);
        *rotations = (double)all;
        if (not_small == large) result = sweep;
        large = not_small;
    }
    free(host);
    return result;
}

// ---- host side of the filtered subspace iteration (see random_rows_kernel) ----------------------------------
constexpr int SUB_CYCLES = 14;
// Products with S before the first Ritz rotation, whose sweeps are the most expensive (9 of 32 from a random block, some 0.2 ms each at 256 rows,
// where a product and one orthonormalisation take 0.4 ms).  Three, five, seven and nine, in ms: 4096 x 4096, rank 128 32.8, 29.9, 30.3, 31.5; rank 256 51.4,
// 52.0, 45.3, 46.9; 1024 x 1024, rank 32 6.5, 6.4, 5.5, 5.7; 2048 x 2048, rank 256 32.6, 28.0, 28.7, 29.1; 4096 x 1024, rank 64 7.5, 7.4, 7.5, 7.6.  One number
// for all: two products more cost 2 to 3 % where they save no cycle of the filter and gain up to 14 % where they do, which the spectrum decides and
// not the size.
constexpr int SUB_POWERS = 7;
constexpr double SUB_SPREAD = 27.6;         // ln 1e12: growth of the largest Ritz direction over the smallest per filter
constexpr double SUB_TOL = 1e-12;           // residual of a leading vector, relative to its Ritz value
constexpr double SUB_DOWNDATE = 1e4;        // spread of the Ritz values up to which S is updated instead of formed again

// vectors of the block for rank r of m: at least twice r, whole block rounds
int subspace_size(int r) { return ((2 * r > r + 64 ? 2 * r : r + 64) + 127) / 128 * 128; }
// taken when the block is at most a quarter of the rows (its buffers then fit one m x m matrix, and the sweeps over all
// rows cost more: 4096 x 4096 with r = 128, 0.78 s of sweeps)
bool subspace_fits(int m, int r) { return subspace_size(r) <= m / 4; }

// the p rows of Z (length L) made orthonormal (passes == 1: nearly, for a block that another product follows); F, inv: p x p scratch each (p >= 64), scratch: `room` doubles
void orthonormalise(double* Z, int p, int L, double* F, double* inv, double* scratch, size_t room, double* thr, unsigned* flag, hipStream_t st, bool clear = true, int passes = 2)
{
    hipLaunchKernelGGL(normalise_rows_kernel, dim3(p), dim3(256), 0, st, Z, L);
    for (int pass = 0; pass < passes; ++pass) {
        gemm((const double*)Z, (long)L, 1L, (const double*)Z, (long)L, 1L, F, (long)p, p, p, L, st, 1.0, 0.0, GM_LOWER, scratch, room);
        cholesky(F, p, 1e-14, thr, flag, inv, st, clear && pass == 0, true);
        for (int j0 = 0; j0 < p; j0 += CH_NB) {
            const int nb = p - j0 < CH_NB ? p - j0 : CH_NB;
            if (j0 > 0)                     // rows j0 .. -= F[j0 .., 0 .. j0) Z[0 .. j0)
                gemm((const double*)(F + (size_t)j0 * p), (long)p, 1L, (const double*)Z, 1L, (long)L, Z + (size_t)j0 * L, (long)L, nb, L, j0, st, -1.0, 1.0);
            // rows j0 .. <- L11^-1 rows, in place (a workgroup reads its 64 columns whole before it writes them)
            gemm((const double*)(inv + (size_t)j0 * CH_NB), (long)CH_NB, 1L, (const double*)(Z + (size_t)j0 * L), 1L, (long)L, Z + (size_t)j0 * L, (long)L, nb, L, nb, st);
        }
    }
}

// S = T T^T (both triangles) of T, m x n
void row_products(const double* T, int m, int n, double* S, hipStream_t st)
{
    gemm(T, (long)n, 1L, T, (long)n, 1L, S, (long)m, m, m, n, st, 1.0, 0.0, GM_LOWER);
    hipLaunchKernelGGL(mirror_kernel, dim3((m + 31) / 32, (m + 31) / 32), dim3(256), 0, st, S, m);
}

// T: m x n.  On success (1) the first p rows of `work` (p x m) are an orthonormal basis that holds the r leading left
// singular vectors of T; 0: not converged or not of rank p (the caller takes another way), < 0: runtime error.
// S: m x m, T1: m x n, XT: r x n, work: room_all >= 3 p m + 3 p^2 doubles, theta / res / lam: p doubles each.  *cycles: filters applied.
int leading_subspace(const double* T, int m, int n, int r, int p, double* S, double* T1, double* XT, double* work, size_t room_all, double* theta, double* res,
                     double* lam, unsigned* flag, double* thr, hipStream_t st, int* cycles)
{
    double* const Z = work;
    double* const Y = Z + (size_t)p * m;
    double* const G = Y + (size_t)p * m;
    double* const R = G + (size_t)p * p;
    double* const F = R + (size_t)p * p;
    double* const U = F + (size_t)p * p;                  // scratch of the rotations and of products in parts: the rest
    const size_t room = room_all - 2 * (size_t)p * m - 3 * (size_t)p * p;
    double* const host = (double*)malloc(sizeof(double) * 2 * p);
    if (!host) return -2;
    double* const h_theta = host;
    double* const h_res = host + p;
    struct Free { double* p; ~Free() { free(p); } } free_host{host};
    double shift = 0.0;                                   // S holds S - shift I
    int nl = 0;                                           // leading rows taken out
    *cycles = 0;
    row_products(T, m, n, S, st);
    auto times_s = [&](const double* A, double* C, int rows, double alpha, double beta) {
        gemm(A, (long)m, 1L, (const double*)S, (long)m, 1L, C, (long)m, rows, m, m, st, alpha, beta, GM_FULL, U, room);
    };
    // Ritz rotation of all p rows: Z <- Ritz vectors (descending), Y <- Z S, theta, residuals, on the host too
    auto ritz = [&]() -> int {
        times_s(Z, Y, p, 1.0, 0.0);
        gemm((const double*)Y, (long)m, 1L, (const double*)Z, (long)m, 1L, F, (long)p, p, p, m, st, 1.0, 0.0, GM_FULL, U, room);
        if (nl > 0)                                       // Y orthogonal to the locked rows: their products with it are F's first columns
            gemm((const double*)(F + (size_t)nl * p), (long)p, 1L, (const double*)Z, 1L, (long)m, Y + (size_t)nl * m, (long)m, p - nl, m, nl, st, -1.0, 1.0);
        hipLaunchKernelGGL(ritz_matrix_kernel, dim3(blocks((size_t)p * p)), dim3(256), 0, st, (const double*)F, G, p, nl, (const double*)theta, shift);
        // G = C C^T; the rows of C^T made orthogonal are the roots of G's eigenvalues times its eigenvectors: no rotations to be
        // gathered, and rows that are unit vectors orthogonal to rounding
        cholesky(G, p, 1e-15, thr, flag, F, st, false);
        hipLaunchKernelGGL(transpose_kernel, dim3((p + 31) / 32, (p + 31) / 32), dim3(256), 0, st, (const double*)G, R, p);
        double rotations = 0;
        const int swept = jacobi_sweeps(R, p, nullptr, p, lam, st, &rotations);
        if (swept < 0) return swept == -1 ? 0 : -2;       // (a runtime error is not "did not settle")
        hipLaunchKernelGGL(row_dot_kernel, dim3(p), dim3(256), 0, st, (const double*)R, (const double*)R, p, lam);
        hipLaunchKernelGGL(sort_rows_kernel, dim3(p), dim3(256), 0, st, (const double*)R, (const double*)lam, p, F, theta);
        gemm((const double*)F, (long)p, 1L, (const double*)Z, 1L, (long)m, U, (long)m, p, m, p, st);
        copy_doubles(U, Z, (size_t)p * m, st);
        gemm((const double*)F, (long)p, 1L, (const double*)Y, 1L, (long)m, U, (long)m, p, m, p, st);
        copy_doubles(U, Y, (size_t)p * m, st);
        hipLaunchKernelGGL(residual_kernel, dim3(p), dim3(256), 0, st, (const double*)Y, (const double*)Z, m, (const double*)theta, shift, res);
        unsigned bad = 1;
        if (hipMemcpyAsync(h_theta, theta, sizeof(double) * p, hipMemcpyDeviceToHost, st) != hipSuccess ||
            hipMemcpyAsync(h_res, res, sizeof(double) * p, hipMemcpyDeviceToHost, st) != hipSuccess ||
            hipMemcpyAsync(&bad, flag, sizeof(bad), hipMemcpyDeviceToHost, st) != hipSuccess || hipStreamSynchronize(st) != hipSuccess)
            return -2;
        return bad == 0 && h_theta[p - 1] > 0.0 && std::isfinite(h_theta[0]) ? 1 : 0;
    };
    hipLaunchKernelGGL(random_rows_kernel, dim3(blocks((size_t)p * m)), dim3(256), 0, st, Y, (size_t)p * m);
    for (int it = 0; it < SUB_POWERS; ++it) {
        times_s(it & 1 ? Z : Y, it & 1 ? Y : Z, p, 1.0, 0.0);
        // (the last one's flag counts: a block that the earlier ones leave nearly dependent, from a spread of S of some 5e7 on, is one that it makes good)
        orthonormalise(it & 1 ? Y : Z, p, m, F, R, U, room, thr, flag, st, it == SUB_POWERS - 1, it == SUB_POWERS - 1 ? 2 : 1);
    }
    static_assert(SUB_POWERS % 2 == 1, "the last product goes to Z");
    int rc = ritz(), stalled = 0;
    double before = 1.0;
    for (int cycle = 0; rc == 1 && cycle < SUB_CYCLES; ++cycle) {
        *cycles = cycle + 1;
        const double a = h_theta[p - 1], x1 = 2.0 * h_theta[nl] / a - 1.0;
        int degree = (int)(SUB_SPREAD / std::acosh(x1 > 1.0 + 1e-9 ? x1 : 1.0 + 1e-9));
        degree = degree < 2 ? 2 : degree > 30 ? 30 : degree;
        hipLaunchKernelGGL(add_diagonal_kernel, dim3(blocks(m)), dim3(256), 0, st, S, m, shift - 0.5 * a);
        shift = 0.5 * a;
        // y_{k+1} = 2 s (2/a) (S - a/2 I) y_k - s_{k-1} s y_{k-1}, scaled so that the direction at x1 keeps its length
        const int rows = p - nl;
        double* y0 = Z + (size_t)nl * m;
        double* y1 = Y + (size_t)nl * m;
        const double sig1 = 1.0 / x1;
        double sig = sig1;
        times_s(y0, y1, rows, sig * 2.0 / a, 0.0);
        for (int k = 2; k <= degree; ++k) {
            const double s2 = 1.0 / (2.0 / sig1 - sig);
            times_s(y1, y0, rows, 2.0 * s2 * 2.0 / a, -sig * s2);
            double* const t = y0;
            y0 = y1;
            y1 = t;
            sig = s2;
        }
        if (y1 != Z + (size_t)nl * m) copy_doubles(y1, Z + (size_t)nl * m, (size_t)rows * m, st);
        if (nl > 0) {                                     // against the rows taken out: z -= (z X^T) X
            gemm((const double*)(Z + (size_t)nl * m), (long)m, 1L, (const double*)Z, (long)m, 1L, F, (long)nl, rows, nl, m, st, 1.0, 0.0, GM_FULL, U, room);
            gemm((const double*)F, (long)nl, 1L, (const double*)Z, 1L, (long)m, Z + (size_t)nl * m, (long)m, rows, m, nl, st, -1.0, 1.0);
        }
        orthonormalise(Z + (size_t)nl * m, rows, m, F, R, U, room, thr, flag, st);
        rc = ritz();
        if (rc != 1) break;
        double worst = 0.0;
        int done = 0;
        for (int i = nl; i < r; ++i) worst = h_res[i] / h_theta[i] > worst ? h_res[i] / h_theta[i] : worst;
        if (getenv("EORA_VERBOSE")) fprintf(stderr, "eora: subspace m=%d p=%d cycle %d degree %d out %d residual %.2e\n", m, p, cycle, degree, nl, worst);
        if (worst <= SUB_TOL) return 1;
        for (done = nl; done < r - 1 && h_res[done] <= SUB_TOL * h_theta[done];) ++done;
        // two cycles that do not halve the residual, with nothing to take out: it does not settle
        const bool lock = done > nl && h_theta[nl] > 4.0 * h_theta[done];
        stalled = lock || worst <= 0.5 * before ? 0 : stalled + 1;
        before = worst;
        if (stalled == 2) return 0;
        if (lock && h_theta[0] > SUB_DOWNDATE * h_theta[r - 1]) {
            // T1 = T - X^T (X T), S = T1 T1^T
            gemm((const double*)Z, (long)m, 1L, T, 1L, (long)n, XT, (long)n, done, n, m, st);
            copy_doubles(T, T1, (size_t)m * n, st);
            gemm((const double*)Z, 1L, (long)m, (const double*)XT, 1L, (long)n, T1, (long)n, m, n, done, st, -1.0, 1.0);
            row_products(T1, m, n, S, st);
            shift = 0.0;
            nl = done;
        } else if (lock) {
            // S -= sum theta_i z_i z_i^T
            copy_doubles(Z + (size_t)nl * m, U, (size_t)(done - nl) * m, st);
            hipLaunchKernelGGL(scale_kernel, dim3(blocks((size_t)(done - nl) * m)), dim3(256), 0, st, U, done - nl, m, (const double*)(theta + nl), 1);
            gemm((const double*)U, 1L, (long)m, (const double*)(Z + (size_t)nl * m), 1L, (long)m, S, (long)m, m, m, done - nl, st, -1.0, 1.0);
            nl = done;
        }
    }
    return rc == 1 ? 0 : rc;
}

inline size_t r256(size_t v) { return (v + 255) & ~(size_t)255; }

struct Layout {
    size_t dW, H, V, T, T0, lam, root, inv, sq, sigma, idx, Ap, Bn, flag, total;
};

Layout layout(int d_in, int d_out, int r)
{
    Layout l;
    size_t o = 0;
    auto take = [&](size_t bytes) {
        const size_t at = o;
        o += r256(bytes);
        return at;
    };
    const size_t big = (size_t)(d_in > d_out ? d_in : d_out);
    l.dW = take(8 * (size_t)d_out * d_in);
    l.H = take(8 * (size_t)d_in * d_in);
    l.V = take(8 * (size_t)d_in * d_in);
    l.T = take(8 * (size_t)d_out * d_in);
    l.T0 = take(8 * (size_t)d_out * d_in);
    l.lam = take(8 * (size_t)d_in);
    l.root = take(8 * (size_t)d_in);
    l.inv = take(8 * (size_t)d_in);
    l.sq = take(8 * big);
    l.sigma = take(8 * (size_t)r);
    l.idx = take(4 * (size_t)r);
    l.Ap = take(8 * (size_t)r * d_in);
    l.Bn = take(8 * (size_t)r * d_out);
    l.flag = take(256);
    l.total = o;
    return l;
}

int g_factors_route = 0;                    // test hook: 0 = Cholesky factor when the Gram matrix allows it, 1 = always the eigendecomposition

int check_shape(int n_tokens, int d_in, int d_out, int r)
{
    if (n_tokens < 1 || d_in < 2 || d_out < 2 || r < 1) return EORA_ERR_SHAPE;
    if (d_in % 2 || d_out % 2 || d_in > MAX_DIM || d_out > MAX_DIM) return EORA_ERR_SHAPE;
    if (r > d_in || r > d_out) return EORA_ERR_SHAPE;
    return EORA_OK;
}

}  // namespace
}  // namespace eora

using namespace eora;

extern "C" void eora_debug_set_factors_route(int route) { g_factors_route = route == 1 ? 1 : 0; }

extern "C" int eora_debug_factors_parts(int M, int N, int K, size_t room)
{
    if (M < 1 || N < 1 || K < 1) return EORA_ERR_SHAPE;
    return gemm_parts(((M + 63) / 64) * ((N + 63) / 64), M, N, K, room);
}

extern "C" int eora_debug_factors_near(int n_tokens) { return near_offsets(n_tokens, 1, sizeof(float)) ? 1 : 0; }

extern "C" size_t eora_factors_workspace_bytes(int d_in, int d_out, int r)
{
    if (check_shape(1, d_in, d_out, r) != EORA_OK) return 0;
    return layout(d_in, d_out, r).total;
}

extern "C" int eora_factors(const void* W_f32, const void* W_hat_f32, const void* Xt_f32, int n_tokens, int d_in, int d_out,
                            int r, double eig_floor, void* B_f64, void* A_f64, void* sigma_f64, void* workspace,
                            size_t workspace_bytes, void* stream, double* stats)
{
    if (!W_f32 || !W_hat_f32 || !Xt_f32 || !B_f64 || !A_f64) return EORA_ERR_NULL;
    const int rc = check_shape(n_tokens, d_in, d_out, r);
    if (rc != EORA_OK) return rc;
    if (!(eig_floor >= 0.0) || eig_floor >= 1.0) return EORA_ERR_VALUE;
    const Layout l = layout(d_in, d_out, r);
    if (!workspace || workspace_bytes < l.total) return EORA_ERR_WORKSPACE;
    if (reinterpret_cast<uintptr_t>(workspace) & 15u) return EORA_ERR_ALIGN;
    hipStream_t st = (hipStream_t)stream;
    char* ws = (char*)workspace;
    double* dW = (double*)(ws + l.dW);
    double* H = (double*)(ws + l.H);
    double* V = (double*)(ws + l.V);
    double* T = (double*)(ws + l.T);
    double* T0 = (double*)(ws + l.T0);
    double* lam = (double*)(ws + l.lam);
    double* root = (double*)(ws + l.root);
    double* inv = (double*)(ws + l.inv);
    double* sq = (double*)(ws + l.sq);
    double* sigma = (double*)(ws + l.sigma);
    int* idx = (int*)(ws + l.idx);
    double* Ap = (double*)(ws + l.Ap);
    double* Bn = (double*)(ws + l.Bn);
    unsigned* flag = (unsigned*)(ws + l.flag);
    double* thr = (double*)(ws + l.flag + 128);
    const float* W = (const float*)W_f32;
    const float* What = (const float*)W_hat_f32;
    const float* Xt = (const float*)Xt_f32;
    const size_t nw = (size_t)d_out * d_in;
    const int k = d_in;

    // steps 1, 2: error and Gram matrix (the factorisation reads the lower triangle only)
    hipLaunchKernelGGL(sub_kernel, dim3(blocks(nw)), dim3(256), 0, st, W, What, dW, nw);
    gemm(Xt, (long)n_tokens, 1L, Xt, (long)n_tokens, 1L, H, (long)k, k, k, n_tokens, st, 1.0, 0.0, g_factors_route == 0 ? GM_LOWER : GM_FULL);

    // Steps 2-4 and 6 by a Cholesky factor.  With X~ X~^T = L L^T, dW L equals dW Q sqrt(Lambda) times an orthogonal
    // matrix on the right, so step 5 finds the same U' and Sigma', and step 6's A = Sigma'^-1 U'^T (dW L) L^-1 is
    // Sigma'^-1 U'^T dW: no inverse at all.  Identical B' and A (up to the signs of the components) whenever no
    // eigenvalue is clamped; taken when every pivot stays above 1e4 * eig_floor * max diag (a Gram matrix that
    // close to singular may have clamped eigenvalues: then the eigendecomposition below decides, as it does when
    // the test hook asks for it).
    bool chol = false;
    if (g_factors_route == 0) {
        hipEvent_t e0 = nullptr, e1 = nullptr;
        const bool timed = stats && hipEventCreate(&e0) == hipSuccess && hipEventCreate(&e1) == hipSuccess;
        if (timed) hipEventRecord(e0, st);
        cholesky(H, k, 1e4 * eig_floor, thr, flag, V, st);
        if (timed) hipEventRecord(e1, st);
        unsigned bad = 1;
        const bool copied = hipMemcpyAsync(&bad, flag, sizeof(bad), hipMemcpyDeviceToHost, st) == hipSuccess &&
                            hipStreamSynchronize(st) == hipSuccess;
        if (timed) {
            float ms = 0;
            hipEventElapsedTime(&ms, e0, e1);
            stats[0] = 0;                        // no sweeps, no rotations, no rows: the Cholesky route
            stats[1] = ms;
            stats[2] = 0;
            stats[3] = 0;
        }
        if (e0) hipEventDestroy(e0);
        if (e1) hipEventDestroy(e1);
        if (!copied) return EORA_ERR_LAUNCH;
        chol = bad == 0;
        if (!chol) gemm(Xt, (long)n_tokens, 1L, Xt, (long)n_tokens, 1L, H, (long)k, k, k, n_tokens, st);      // the Gram matrix again
    }
    int sweeps = 0;
    if (!chol) {
        // step 2: eigenvectors as the rows of V
        hipLaunchKernelGGL(identity_kernel, dim3(blocks((size_t)k * k)), dim3(256), 0, st, V, k);
        sweeps = jacobi(H, k, V, k, sq, st, stats);
        if (sweeps < 0) return sweeps == -1 ? EORA_ERR_NOT_CONVERGED : EORA_ERR_LAUNCH;
        hipLaunchKernelGGL(row_dot_kernel, dim3(k), dim3(256), 0, st, H, V, k, lam);
        // step 3: sqrt(Lambda), with eigenvalues below eig_floor * max raised to it
        hipLaunchKernelGGL(eig_roots_kernel, dim3(1), dim3(1024), 0, st, lam, k, eig_floor, root, inv);
    }

    const bool by_rows = d_out <= d_in;         // which side of dW' has fewer rows to rotate
    const int m = by_rows ? d_out : k, n = by_rows ? k : d_out;       // T: m rows of length n, m <= n
    // step 4: T = dW' (by_rows) or its transpose
    if (by_rows) {
        if (chol) {
            // T = dW L (d_out x k): T[o][j] = sum_i dW[o][i] L[i][j]
            gemm(dW, (long)k, 1L, H, 1L, (long)k, T, (long)k, d_out, k, k, st, 1.0, 0.0, GM_B_LOWER);
        } else {
            // T[o][j] = root[j] * sum_i dW[o][i] V[j][i]
            gemm(dW, (long)k, 1L, V, (long)k, 1L, T, (long)k, d_out, k, k, st);
            hipLaunchKernelGGL(scale_kernel, dim3(blocks(nw)), dim3(256), 0, st, T, d_out, k, root, 0);
        }
    } else {
        if (chol) {
            // T = (dW L)^T (k x d_out): T[j][o] = sum_i L[i][j] dW[o][i]
            gemm(H, 1L, (long)k, dW, (long)k, 1L, T, (long)d_out, k, d_out, k, st, 1.0, 0.0, GM_A_LOWER);
        } else {
            // T[j][o] = root[j] * sum_i V[j][i] dW[o][i]
            gemm(V, (long)k, 1L, dW, (long)k, 1L, T, (long)d_out, k, d_out, k, st);
            hipLaunchKernelGGL(scale_kernel, dim3(blocks(nw)), dim3(256), 0, st, T, k, d_out, root, 1);
        }
    }

    // Step 5 on a square factor when T is at least twice as long as it has rows (Cholesky route only; H and V are
    // free by now): with T T^T = C C^T (Cholesky, C lower), T = C F^T for an F with orthonormal columns, so T and C
    // have the same singular values and left singular vectors w_i; the sweeps rotate the m rows of C^T (length m
    // instead of n) to sigma_i w_i^T, and w_i^T T is the row sigma_i z_i^T the sweeps over T itself would have
    // ended with.  The r largest components are accurate to the rounding of T T^T relative to sigma_1^2; a T of
    // rank below m (an error of low rank) has no such factor: then, as before, the rows of T are rotated.
    bool square = false;
    // r well below m: the leading subspace instead of all m components (H and V are free by now).  0: it did not settle
    // (no gap behind the block, or an error of rank below the block's size): then as for larger ranks.
    int sub = 0;
    const int p = subspace_size(r);
    if (chol && subspace_fits(m, r)) {
        hipEvent_t e0 = nullptr, e1 = nullptr;
        const bool timed = stats && hipEventCreate(&e0) == hipSuccess && hipEventCreate(&e1) == hipSuccess;
        if (timed) hipEventRecord(e0, st);
        int cycles = 0;
        sub = leading_subspace(T, m, n, r, p, H, T0, by_rows ? Ap : Bn, V, (size_t)k * k, lam, root, inv, flag, thr, st, &cycles);
        if (stats) stats[0] = sub == 1 ? cycles : -cycles;
        if (sub == 1) {
            gemm((const double*)V, (long)m, 1L, (const double*)T, 1L, (long)n, T0, (long)n, p, n, m, st, 1.0, 0.0, GM_FULL, H, (size_t)k * k);      // Z T
            sweeps = jacobi(T0, n, nullptr, p, sq, st, stats ? stats + 4 : nullptr);
            if (sweeps < 0) return sweeps == -1 ? EORA_ERR_NOT_CONVERGED : EORA_ERR_LAUNCH;
            hipLaunchKernelGGL(row_dot_kernel, dim3(p), dim3(256), 0, st, T0, T0, n, sq);
            hipLaunchKernelGGL(top_rows_kernel, dim3(blocks(p)), dim3(256), 0, st, sq, p, r, idx, sigma);
            if (stats) stats[2] = n;
        }
        if (timed) {
            float ms = 0;
            hipEventRecord(e1, st);
            hipEventSynchronize(e1);
            hipEventElapsedTime(&ms, e0, e1);
            stats[5] = ms;
        }
        if (e0) hipEventDestroy(e0);
        if (e1) hipEventDestroy(e1);
        if (sub < 0) return EORA_ERR_LAUNCH;
    }
    if (chol && !sub && n >= 2 * m) {
        gemm(T, (long)n, 1L, T, (long)n, 1L, H, (long)m, m, m, n, st, 1.0, 0.0, GM_LOWER);
        cholesky(H, m, 1e-14, thr, flag, V, st);
        unsigned bad = 1;
        if (hipMemcpyAsync(&bad, flag, sizeof(bad), hipMemcpyDeviceToHost, st) != hipSuccess || hipStreamSynchronize(st) != hipSuccess)
            return EORA_ERR_LAUNCH;
        square = bad == 0;
    }
    const double* Tkeep = T;                    // T as step 4 left it
    if (sub) {
        // rows idx[i] of T0: sigma_i z_i^T
    } else if (square) {
        double* Y = V;                          // C^T
        hipLaunchKernelGGL(transpose_kernel, dim3((m + 31) / 32, (m + 31) / 32), dim3(256), 0, st, (const double*)H, Y, m);
        sweeps = jacobi(Y, m, nullptr, m, sq, st, stats ? stats + 4 : nullptr);
        if (sweeps < 0) return sweeps == -1 ? EORA_ERR_NOT_CONVERGED : EORA_ERR_LAUNCH;
        hipLaunchKernelGGL(row_dot_kernel, dim3(m), dim3(256), 0, st, Y, Y, m, sq);
        hipLaunchKernelGGL(top_rows_kernel, dim3(blocks(m)), dim3(256), 0, st, sq, m, r, idx, sigma);
        // the r rows sigma_i z_i^T = w_i^T T, into T0 (r x n)
        double* Wr = by_rows ? Bn : Ap;         // r x m unit rows w_i^T (Bn: r x d_out, Ap: r x k)
        hipLaunchKernelGGL(gather_rows_kernel, dim3(blocks((size_t)r * m)), dim3(256), 0, st, Y, m, idx, sigma, -1, Wr, r);
        gemm(Wr, (long)m, 1L, T, 1L, (long)n, T0, (long)n, r, n, m, st);
        hipLaunchKernelGGL(iota_kernel, dim3(blocks(r)), dim3(256), 0, st, idx, r);
        if (stats) stats[2] = m;                // (Cholesky route: the length of the rows the SVD's sweeps rotated)
    } else {
        copy_doubles(T, T0, nw, st);
        Tkeep = T0;
        // step 5: rows of T -> sigma_i z_i^T
        sweeps = jacobi(T, n, nullptr, m, sq, st, stats ? stats + 4 : nullptr);
        if (sweeps < 0) return sweeps == -1 ? EORA_ERR_NOT_CONVERGED : EORA_ERR_LAUNCH;
        hipLaunchKernelGGL(row_dot_kernel, dim3(m), dim3(256), 0, st, T, T, n, sq);
        hipLaunchKernelGGL(top_rows_kernel, dim3(blocks(m)), dim3(256), 0, st, sq, m, r, idx, sigma);
        if (stats && chol) stats[2] = n;
    }
    // (the Gram matrix, its factor, S or the square factor in H are done with: room for the parts of the products below)
    const double* Tc = sub || square ? T0 : T;  // rows idx[i]: sigma_i z_i^T
    if (by_rows) {
        // z_i = v_i: A' = rows of V'^T; B' = U' Sigma' = dW' A'^T
        hipLaunchKernelGGL(gather_rows_kernel, dim3(blocks((size_t)r * k)), dim3(256), 0, st, Tc, k, idx, sigma, -1, Ap, r);
        gemm(Tkeep, (long)k, 1L, Ap, (long)k, 1L, (double*)B_f64, (long)r, d_out, r, k, st, 1.0, 0.0, GM_FULL, H, (size_t)k * k);
        // Cholesky route, step 6: A = Sigma'^-2 B'^T dW
        if (chol) hipLaunchKernelGGL(scaled_transpose_kernel, dim3(blocks((size_t)r * d_out)), dim3(256), 0, st, (const double*)B_f64, sigma, d_out, r, Bn);
    } else {
        // z_i = u_i: the columns of B' are sigma_i u_i
        hipLaunchKernelGGL(gather_rows_transposed_kernel, dim3(blocks((size_t)r * d_out)), dim3(256), 0, st, Tc, d_out, idx,
                           (double*)B_f64, r);
        // A' = Sigma'^-1 U'^T dW' : A'[i][j] = sum_o (sigma_i u_i[o] / sigma_i^2) dW'[o][j]
        hipLaunchKernelGGL(gather_rows_kernel, dim3(blocks((size_t)r * d_out)), dim3(256), 0, st, Tc, d_out, idx, sigma, -2, Bn,
                           r);
        if (!chol) gemm(Bn, (long)d_out, 1L, Tkeep, (long)d_out, 1L, Ap, (long)k, r, k, d_out, st, 1.0, 0.0, GM_FULL, H, (size_t)k * k);
    }
    if (chol) {
        // step 6 without an inverse: A[i][j] = sum_o (sigma_i u_i[o] / sigma_i^2) dW[o][j]
        gemm(Bn, (long)d_out, 1L, dW, 1L, (long)k, (double*)A_f64, (long)k, r, k, d_out, st, 1.0, 0.0, GM_FULL, H, (size_t)k * k);
    } else {
        // step 6: A = A' sqrt(Lambda)^-1 Q^T : A[i][j] = sum_e A'[i][e] inv[e] V[e][j]
        hipLaunchKernelGGL(scale_kernel, dim3(blocks((size_t)r * k)), dim3(256), 0, st, Ap, r, k, inv, 0);
        gemm(Ap, (long)k, 1L, V, 1L, (long)k, (double*)A_f64, (long)k, r, k, k, st, 1.0, 0.0, GM_FULL, H, (size_t)k * k);
    }
    if (sigma_f64) hipLaunchKernelGGL(copy_kernel, dim3(blocks(r)), dim3(256), 0, st, sigma, (double*)sigma_f64, (size_t)r);
    if (hipGetLastError() != hipSuccess) return EORA_ERR_LAUNCH;
    if (hipStreamSynchronize(st) != hipSuccess) return EORA_ERR_LAUNCH;
    return EORA_OK;
}

extern "C" int eora_factors_store_f16(const void* B_f64, const void* A_f64, int d_in, int d_out, int r, int balance,
                                      void* A_tiles, void* B_tiles, void* scratch, size_t scratch_bytes, void* stream)
{
    if (!B_f64 || !A_f64 || !A_tiles || !B_tiles) return EORA_ERR_NULL;
    if (d_in <= 0 || d_out <= 0 || r <= 0 || d_in % 32 || d_out % 16 || r % 32) return EORA_ERR_SHAPE;
    if ((reinterpret_cast<uintptr_t>(A_tiles) | reinterpret_cast<uintptr_t>(B_tiles) | reinterpret_cast<uintptr_t>(B_f64) |
         reinterpret_cast<uintptr_t>(A_f64)) & 15u)
        return EORA_ERR_ALIGN;
    double* s = nullptr;
    if (balance) {
        if (!scratch || scratch_bytes < sizeof(double) * (size_t)r) return EORA_ERR_WORKSPACE;
        if (reinterpret_cast<uintptr_t>(scratch) & 15u) return EORA_ERR_ALIGN;
        s = (double*)scratch;
    }
    hipStream_t st = (hipStream_t)stream;
    if (s) hipLaunchKernelGGL(balance_kernel, dim3(r), dim3(256), 0, st, (const double*)B_f64, (const double*)A_f64, d_in, d_out, r, s);
    hipLaunchKernelGGL(store_f16_tiles_kernel, dim3(blocks((size_t)r * d_in / 8)), dim3(256), 0, st, (const double*)A_f64, r, d_in,
                       (const double*)s, 1, (_Float16*)A_tiles);
    hipLaunchKernelGGL(store_f16_tiles_kernel, dim3(blocks((size_t)d_out * r / 8)), dim3(256), 0, st, (const double*)B_f64, d_out, r,
                       (const double*)s, 0, (_Float16*)B_tiles);
    if (hipGetLastError() != hipSuccess) return EORA_ERR_LAUNCH;
    return EORA_OK;
}

extern "C" int eora_factors_store_q(const void* B_f64, const void* A_f64, int d_in, int d_out, int r, int ab_bits, int balance,
                                    void* A_q, void* A_scales, void* B_q, void* B_scales, void* scratch, size_t scratch_bytes,
                                    void* stream)
{
    if (!B_f64 || !A_f64 || !A_q || !A_scales || !B_q || !B_scales) return EORA_ERR_NULL;
    if (ab_bits != 4 && ab_bits != 3) return EORA_ERR_UNSUPPORTED;
    if (d_in <= 0 || d_out <= 0 || r <= 0 || d_in % 128 || d_out % 16) return EORA_ERR_SHAPE;
    if (!(r % 128 == 0 || (ab_bits == 4 && r == 64))) return EORA_ERR_SHAPE;
    if ((reinterpret_cast<uintptr_t>(A_q) | reinterpret_cast<uintptr_t>(B_q) | reinterpret_cast<uintptr_t>(A_scales) |
         reinterpret_cast<uintptr_t>(B_scales) | reinterpret_cast<uintptr_t>(B_f64) | reinterpret_cast<uintptr_t>(A_f64)) & 15u)
        return EORA_ERR_ALIGN;
    double* s = nullptr;
    if (balance) {
        if (!scratch || scratch_bytes < sizeof(double) * (size_t)r) return EORA_ERR_WORKSPACE;
        if (reinterpret_cast<uintptr_t>(scratch) & 15u) return EORA_ERR_ALIGN;
        s = (double*)scratch;
    }
    hipStream_t st = (hipStream_t)stream;
    const double* A = (const double*)A_f64;
    const double* B = (const double*)B_f64;
    if (s) hipLaunchKernelGGL(balance_kernel, dim3(r), dim3(256), 0, st, B, A, d_in, d_out, r, s);
    const dim3 ga((r / 16) * (d_in / 128)), gb((d_out / 16) * (r / (r == 64 ? 64 : 128)));
    if (ab_bits == 4) {
        hipLaunchKernelGGL((store_q_tiles_kernel<4, 128>), ga, dim3(64), 0, st, A, r, d_in, (const double*)s, 1, (uint32_t*)A_q, (_Float16*)A_scales);
        if (r == 64)
            hipLaunchKernelGGL((store_q_tiles_kernel<4, 64>), gb, dim3(64), 0, st, B, d_out, r, (const double*)s, 0, (uint32_t*)B_q, (_Float16*)B_scales);
        else
            hipLaunchKernelGGL((store_q_tiles_kernel<4, 128>), gb, dim3(64), 0, st, B, d_out, r, (const double*)s, 0, (uint32_t*)B_q, (_Float16*)B_scales);
    } else {
        hipLaunchKernelGGL((store_q_tiles_kernel<3, 128>), ga, dim3(64), 0, st, A, r, d_in, (const double*)s, 1, (uint32_t*)A_q, (_Float16*)A_scales);
        hipLaunchKernelGGL((store_q_tiles_kernel<3, 128>), gb, dim3(64), 0, st, B, d_out, r, (const double*)s, 0, (uint32_t*)B_q, (_Float16*)B_scales);
    }
    if (hipGetLastError() != hipSuccess) return EORA_ERR_LAUNCH;
    return EORA_OK;
}
