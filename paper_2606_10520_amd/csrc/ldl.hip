// Block LDL^T factorisation of the layer Hessian on gfx950 (Sec. 3.2.2,
// Eq. 7): H = U D U^T with U unit upper block-triangular (4 x 4 identity
// blocks on the diagonal, zeros below them) and D block diagonal with 4 x 4
// blocks -- the factor whose off-diagonal entries are LDLQ's feedback
// coefficients.  All arithmetic in fp64.
//
// With U unit upper triangular the factorisation runs from the last column
// block to the first (the last pivot is H's own last diagonal block).  With
// S the part of H not yet factorised (its upper triangle held in U's own
// buffer), one 4 x 4 pivot block j gives
//     D_j = S_jj,   U[0:j, j] = S[0:j, j] D_j^-1,
//     S[0:j, 0:j] -= U[0:j, j] D_j U[0:j, j]^T.
// Blocked over panels of 64 columns (16 pivot blocks), right to left, two
// launches per panel:
//  1. strip: every row r above the panel solves w U_pp^T = S[r, panel]
//     (U_pp the panel's factor, unit upper: a back substitution over its
//     pivot blocks) and stores w and U[r, panel] = w D_p^-1, one wavefront
//     per row, lane c = panel column c;
//  2. trailing: S[a][b] -= sum_k W[a][k] U[b][k] over the panel's 64
//     columns, for a <= b above the panel (64 x 64 tiles of the upper
//     triangle on the fp64 matrix cores).  The workgroup of the next panel's
//     diagonal tile, the first of the launch, keeps its tile in registers and
//     factorises it pivot block by pivot block while the others update
//     theirs (the panel's serial part: as a launch of its own it was 1.4 of
//     3.1 ms at K = 4096).
// K = 4096, MI355X: 1.9 ms (3.14 before).  A diagonal block alone takes 14 us
// (23 with its 64 x 64 block in LDS and two barriers per pivot); a trailing
// launch 42 to 17 us, the lower end set by the pivots; a strip 5 to 8 us.
// Error against an 80-bit factorisation (K = 128 to 1024, twelve Hessians of
// condition about 1e5): 9e-15 to 1.1e-13, as before.
// Every pivot block is checked for positive definiteness (its leading
// principal minors); the first failure is reported through `info`.
#include "common.hpp"

namespace unisvq {
namespace {

constexpr int kLdlP = 64;          // panel width (16 pivot blocks of 4)
constexpr int kLdlPitch = kLdlP + 1;  // LDS row pitch (doubles) of the diagonal block

__device__ inline double lane_f64(double v, int src) {
    const uint2 u = __builtin_bit_cast(uint2, v);
    return __builtin_bit_cast(double, uint2{static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(u.x), src)),
                                            static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(u.y), src))});
}

// U = upper triangle of H (a <= b), zeros below; info = 0.  Two elements per
// thread (K is even).  In place when U == H: each element is read and
// written by the same thread.
__global__ __launch_bounds__(256) void ldl_init_kernel(const double* H, double* U, int64_t K, int32_t* info) {
    const int64_t e = (static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x) * 2;
    if (e == 0 && info) *info = 0;
    if (e >= K * K) return;
    const int64_t a = e / K, b = e - a * K;
    double2 h = double2{0.0, 0.0};
    if (a <= b + 1) h = *reinterpret_cast<const double2*>(H + e);
    *reinterpret_cast<double2*>(U + e) = double2{a <= b ? h.x : 0.0, a <= b + 1 ? h.y : 0.0};
}

// a b - c d to within two roundings of the result (Kahan): the fma recovers the
// rounding error of c d.  The minors of a pivot block whose columns share a
// common component cancel to a small part of their products.
__device__ inline double det2(double a, double b, double c, double d) {
    const double w = c * d;
    return fma(a, b, -w) + fma(-c, d, w);
}

// Inverse of a 4 x 4 matrix by Laplace expansion along its first two rows
// (complementary 2 x 2 minors: s_ of rows 0, 1, c_ of rows 2, 3), every
// index fixed at compile time; returns the determinant.
__device__ inline double inverse4(const double (&m)[4][4], double (&b)[4][4]) {
    const double s0 = det2(m[0][0], m[1][1], m[1][0], m[0][1]), s1 = det2(m[0][0], m[1][2], m[1][0], m[0][2]);
    const double s2 = det2(m[0][0], m[1][3], m[1][0], m[0][3]), s3 = det2(m[0][1], m[1][2], m[1][1], m[0][2]);
    const double s4 = det2(m[0][1], m[1][3], m[1][1], m[0][3]), s5 = det2(m[0][2], m[1][3], m[1][2], m[0][3]);
    const double c5 = det2(m[2][2], m[3][3], m[3][2], m[2][3]), c4 = det2(m[2][1], m[3][3], m[3][1], m[2][3]);
    const double c3 = det2(m[2][1], m[3][2], m[3][1], m[2][2]), c2 = det2(m[2][0], m[3][3], m[3][0], m[2][3]);
    const double c1 = det2(m[2][0], m[3][2], m[3][0], m[2][2]), c0 = det2(m[2][0], m[3][1], m[3][0], m[2][1]);
    const double det = s0 * c5 - s1 * c4 + s2 * c3 + s3 * c2 - s4 * c1 + s5 * c0;
    const double r = 1.0 / det;
    b[0][0] = (m[1][1] * c5 - m[1][2] * c4 + m[1][3] * c3) * r;
    b[0][1] = (-m[0][1] * c5 + m[0][2] * c4 - m[0][3] * c3) * r;
    b[0][2] = (m[3][1] * s5 - m[3][2] * s4 + m[3][3] * s3) * r;
    b[0][3] = (-m[2][1] * s5 + m[2][2] * s4 - m[2][3] * s3) * r;
    b[1][0] = (-m[1][0] * c5 + m[1][2] * c2 - m[1][3] * c1) * r;
    b[1][1] = (m[0][0] * c5 - m[0][2] * c2 + m[0][3] * c1) * r;
    b[1][2] = (-m[3][0] * s5 + m[3][2] * s2 - m[3][3] * s1) * r;
    b[1][3] = (m[2][0] * s5 - m[2][2] * s2 + m[2][3] * s1) * r;
    b[2][0] = (m[1][0] * c4 - m[1][1] * c2 + m[1][3] * c0) * r;
    b[2][1] = (-m[0][0] * c4 + m[0][1] * c2 - m[0][3] * c0) * r;
    b[2][2] = (m[3][0] * s4 - m[3][1] * s2 + m[3][3] * s0) * r;
    b[2][3] = (-m[2][0] * s4 + m[2][1] * s2 - m[2][3] * s0) * r;
    b[3][0] = (-m[1][0] * c3 + m[1][1] * c1 - m[1][2] * c0) * r;
    b[3][1] = (m[0][0] * c3 - m[0][1] * c1 + m[0][2] * c0) * r;
    b[3][2] = (-m[3][0] * s3 + m[3][1] * s1 - m[3][2] * s0) * r;
    b[3][3] = (m[2][0] * s3 - m[2][1] * s1 + m[2][2] * s0) * r;
    return det;
}

// Rows r < c0 against the panel [c0, c0 + 64): w U_pp^T = S[r, panel]
// (back substitution, the last pivot block first), W[r] = w,
// U[r, panel] = w D_p^-1.  One wavefront per row, lane c = column c0 + c.
__global__ __launch_bounds__(256) void ldl_strip_kernel(double* U, int64_t K, int64_t c0, const double* dinv,
                                                        double* W) {
    __shared__ double Up[kLdlP * kLdlPitch];
    __shared__ double Di[16 * 16];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const double* const blk = U + c0 * K + c0;
    {
        double v[kLdlP / 4];
#pragma unroll
        for (int k = 0; k < kLdlP / 4; ++k) v[k] = blk[(wave + 4 * k) * K + lane];
        const double di = dinv[t];
#pragma unroll
        for (int k = 0; k < kLdlP / 4; ++k) Up[(wave + 4 * k) * kLdlPitch + lane] = v[k];
        Di[t] = di;
    }
    __syncthreads();
    const int b = lane >> 2;  // the lane's pivot block
    for (int64_t r = static_cast<int64_t>(blockIdx.x) * 4 + wave; r < c0; r += static_cast<int64_t>(gridDim.x) * 4) {
        double s = U[r * K + c0 + lane];
        for (int jb = kLdlP / 4 - 1; jb >= 1; --jb) {
            // block jb is final: remove its part from the lanes of the blocks before it
            const double w0 = lane_f64(s, 4 * jb), w1 = lane_f64(s, 4 * jb + 1);
            const double w2 = lane_f64(s, 4 * jb + 2), w3 = lane_f64(s, 4 * jb + 3);
            if (b < jb) {
                const double* const up = Up + lane * kLdlPitch + 4 * jb;
                double acc = w0 * up[0];
                acc = fma(w1, up[1], acc);
                acc = fma(w2, up[2], acc);
                acc = fma(w3, up[3], acc);
                s -= acc;
            }
        }
        W[r * kLdlP + lane] = s;
        // u = w D^-1 within the lane's pivot block
        double u = 0.0;
#pragma unroll
        for (int n = 0; n < 4; ++n) u = fma(__shfl(s, (lane & ~3) + n, 64), Di[b * 16 + n * 4 + (lane & 3)], u);
        U[r * K + c0 + lane] = u;
    }
}

constexpr int kLdlMPitch = kLdlP + 4;
typedef double f64x4 __attribute__((ext_vector_type(4)));

// (by value: a conditional on array elements themselves puts the array in memory)
__device__ inline double pick(bool c, double a, double b) { return c ? a : b; }

// Pivot blocks of tile column TC (panel columns 16 TC .. 16 TC + 15), the last
// first.  Wavefront w holds S's rows 16 w .. 16 w + 15 as tiles acc[tj] of
// columns 16 tj in matrix-core result layout; wavefronts above TC have no rows
// left.  Per pivot block at column a:
//  * the column strip S[0:a+4, a:a+4] goes to P (one 64 x 4 buffer per pivot
//    block, so one barrier each);
//  * every lane inverts D itself; lane (i, k) forms u[i][k] = sum_n S[i][n]
//    D^-1[n][k], which is the A operand, and P's rows are the B operand, of
//    S -= u S[., a:a+4]^T (each lane taking only its column of the inverse,
//    from four cofactors of a permuted D, was shorter but up to six times
//    less accurate at K = 128);
//  * u and the identity block go to U.
// Only S[r][c] with r <= c < a is live; everything else (what lies below the
// diagonal, columns a and beyond) takes whatever it gets and feeds only
// entries of the same kind.
template <int TC>
__device__ inline void pivots(f64x4 (&acc)[4], double (*P)[kLdlP * 4], int w, int lane, double* blk, int64_t K) {
    const int li = lane & 15, lk = lane >> 4;
#pragma clang loop unroll(disable)
    for (int jq = 3; jq >= 0; --jq) {
        const int a = 16 * TC + 4 * jq;
        double* const p = P[4 * TC + jq];
        if (w <= TC && (li >> 2) == jq) {
#pragma unroll
            for (int v = 0; v < 4; ++v) p[(16 * w + lk + 4 * v) * 4 + (li & 3)] = acc[TC][v];
        }
        __syncthreads();
        if (w <= TC) {  // uniform
            double d[4][4], inv[4][4], b[TC + 1];
#pragma unroll
            for (int n = 0; n < 4; ++n)
#pragma unroll
                for (int m = 0; m < 4; ++m) d[n][m] = p[4 * (a + (n < m ? n : m)) + (n < m ? m : n)];
            double q[4];
#pragma unroll
            for (int n = 0; n < 4; ++n) q[n] = p[4 * (16 * w + li) + n];
#pragma unroll
            for (int tj = 0; tj <= TC; ++tj) b[tj] = p[4 * (16 * tj + li) + lk];
            inverse4(d, inv);
            double u = 0.0;
#pragma unroll
            for (int n = 0; n < 4; ++n) {
                u = fma(q[n], pick(lk & 2, pick(lk & 1, inv[n][3], inv[n][2]), pick(lk & 1, inv[n][1], inv[n][0])), u);
            }
#pragma unroll
            for (int tj = 0; tj <= TC; ++tj)
                if (tj >= w) acc[tj] -= __builtin_amdgcn_mfma_f64_16x16x4f64(u, b[tj], f64x4{0.0, 0.0, 0.0, 0.0}, 0, 0, 0);
            const int r = 16 * w + li;
            if (r < a + 4) blk[r * K + a + lk] = r < a ? u : (r - a == lk ? 1.0 : 0.0);
        }
    }
}

// The panel's 64 x 64 diagonal block at c0, in acc as above: its factor to U,
// the pivot blocks to D, their inverses to dinv, and the check of positive
// definiteness (sixteen threads after the pivots, from the strips in P).
__device__ inline void factorise(f64x4 (&acc)[4], double (*P)[kLdlP * 4], double* U, int64_t K, int64_t c0, double* D,
                                 int32_t* info, double* dinv) {
    const int t = threadIdx.x, lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6);
    double* const blk = U + c0 * K + c0;
    pivots<3>(acc, P, w, lane, blk, K);
    pivots<2>(acc, P, w, lane, blk, K);
    pivots<1>(acc, P, w, lane, blk, K);
    pivots<0>(acc, P, w, lane, blk, K);
    if (t < 64) {  // wavefront 0; thread jb < 16 takes pivot block jb
        const int jb = t & 15;
        double d[4][4], inv[4][4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) d[i][j] = P[jb][(4 * jb + (i < j ? i : j)) * 4 + (i < j ? j : i)];
        const double det = inverse4(d, inv);
        const double m2 = d[0][0] * d[1][1] - d[1][0] * d[0][1];
        const double m3 = d[0][0] * (d[1][1] * d[2][2] - d[1][2] * d[2][1]) -
                          d[0][1] * (d[1][0] * d[2][2] - d[1][2] * d[2][0]) +
                          d[0][2] * (d[1][0] * d[2][1] - d[1][1] * d[2][0]);
        const bool ok = d[0][0] > 0.0 && m2 > 0.0 && m3 > 0.0 && det > 0.0;  // false on NaN
        const uint32_t bad = static_cast<uint32_t>(__ballot(!ok)) & 0xffffu;
        if (t < 16) {
#pragma unroll
            for (int i = 0; i < 16; ++i) dinv[jb * 16 + i] = inv[i >> 2][i & 3];
            if (D) {
#pragma unroll
                for (int i = 0; i < 16; ++i) D[(c0 / 4 + jb) * 16 + i] = d[i >> 2][i & 3];
            }
            // the first to fail is the highest: the last pivot goes first
            if (t == 0 && bad && info && *info == 0) *info = static_cast<int32_t>(c0 / 4 + 32 - __clz(static_cast<int>(bad)));
        }
    }
}

// The last panel's diagonal block, which no trailing update comes before.
__global__ __launch_bounds__(256) void ldl_diag_kernel(double* U, int64_t K, int64_t c0, double* D, int32_t* info,
                                                       double* dinv) {
    __shared__ double P[16][kLdlP * 4];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    f64x4 acc[4];
#pragma unroll
    for (int tj = 0; tj < 4; ++tj)
#pragma unroll
        for (int v = 0; v < 4; ++v)
            acc[tj][v] = U[(c0 + 16 * w + (lane >> 4) + 4 * v) * K + c0 + 16 * tj + (lane & 15)];
    factorise(acc, P, U, K, c0, D, info, dinv);
}

// S[a][b] -= sum_k W[a][k] U[b][c0 + k] for a <= b < c0: one 64 x 64 tile of
// rows 64 ta, columns 64 tb, ta <= tb, per workgroup, on the fp64 matrix
// cores, the last diagonal tile (the next panel's, which goes on to be
// factorised) first.  Both 64 x 64 operands are staged row-major in LDS (pitch
// 68 doubles: an operand read touches every bank the minimum number of
// times); wavefront w computes rows 16 w .. 16 w + 15 as four 16 x 16 blocks
// over 16 steps of 4 columns of k.  Operand lanes: A[i][k] at lane i + 16 k,
// B[k][j] at lane j + 16 k; result D[i][j] at lane j + 16 (i % 4), item i / 4.
struct TrailLds {
    double Ws[kLdlP * kLdlMPitch];  // [row][k]
    double Us[kLdlP * kLdlMPitch];  // [column][k]
};
static_assert(sizeof(TrailLds) >= 16 * kLdlP * 4 * 8, "the pivot strips reuse the operands' LDS");

__global__ __launch_bounds__(256) void ldl_trailing_kernel(double* U, int64_t K, int64_t c0, const double* W, double* D,
                                                           int32_t* info, double* dinv) {
    __shared__ __attribute__((aligned(16))) TrailLds sh;
    // tile number counted from the last diagonal tile down: tb by rows of the triangle
    const int nt = static_cast<int>(c0 / kLdlP);
    const int id = nt * (nt + 1) / 2 - 1 - static_cast<int>(blockIdx.x);
    int tb = static_cast<int>((sqrtf(8.0f * static_cast<float>(id) + 1.0f) - 1.0f) * 0.5f);
    while (tb * (tb + 1) / 2 > id) --tb;
    while ((tb + 1) * (tb + 2) / 2 <= id) ++tb;
    tb = __builtin_amdgcn_readfirstlane(tb);
    const int ta = __builtin_amdgcn_readfirstlane(id - tb * (tb + 1) / 2);
    const int t = threadIdx.x, lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6);
    const int64_t a0 = static_cast<int64_t>(ta) * kLdlP, b0 = static_cast<int64_t>(tb) * kLdlP;
    const int li = lane & 15, lk = lane >> 4;
    // this lane's 16 outputs, read now (every one in bounds: the tile lies
    // above row c0) and written back after the products
    double old[4][4];
    double* const out = U + (a0 + 16 * w + lk) * K + b0 + li;
#pragma unroll
    for (int tj = 0; tj < 4; ++tj)
#pragma unroll
        for (int v = 0; v < 4; ++v) old[tj][v] = out[4 * v * K + 16 * tj];
    {
        // the operands, 16 + 16 coalesced loads per thread in flight at once
        // (row rq + 4k, column c of each 64 x 64 operand)
        const int c = t & 63, rq = t >> 6;
        double wv[kLdlP / 4], uv[kLdlP / 4];
#pragma unroll
        for (int k = 0; k < kLdlP / 4; ++k) {
            wv[k] = W[(a0 + rq + 4 * k) * kLdlP + c];
            uv[k] = U[(b0 + rq + 4 * k) * K + c0 + c];
        }
#pragma unroll
        for (int k = 0; k < kLdlP / 4; ++k) {
            sh.Ws[(rq + 4 * k) * kLdlMPitch + c] = wv[k];
            sh.Us[(rq + 4 * k) * kLdlMPitch + c] = uv[k];
        }
    }
    __syncthreads();
    f64x4 acc[4];
#pragma unroll
    for (int tj = 0; tj < 4; ++tj) acc[tj] = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int s = 0; s < kLdlP / 4; ++s) {
        const double av = sh.Ws[(16 * w + li) * kLdlMPitch + 4 * s + lk];
#pragma unroll
        for (int tj = 0; tj < 4; ++tj)
            acc[tj] = __builtin_amdgcn_mfma_f64_16x16x4f64(av, sh.Us[(16 * tj + li) * kLdlMPitch + 4 * s + lk], acc[tj],
                                                           0, 0, 0);
    }
#pragma unroll
    for (int tj = 0; tj < 4; ++tj)
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[tj][v] = old[tj][v] - acc[tj][v];
    if (blockIdx.x == 0) {  // uniform: the next panel's diagonal block
        __syncthreads();    // the operands' LDS becomes the pivot strips'
        factorise(acc, reinterpret_cast<double(*)[kLdlP * 4]>(&sh), U, K, b0, D, info, dinv);
        return;
    }
#pragma unroll
    for (int tj = 0; tj < 4; ++tj)
#pragma unroll
        for (int v = 0; v < 4; ++v)
            if (ta < tb || 16 * w + lk + 4 * v <= 16 * tj + li) out[4 * v * K + 16 * tj] = acc[tj][v];
}

}  // namespace

size_t ldl_workspace_bytes(int64_t K) {
    return static_cast<size_t>(K) * kLdlP * 8 + 16 * 16 * 8;
}

hipError_t launch_ldl(int64_t K, const double* H, double* U, double* D, int32_t* info, void* workspace,
                      hipStream_t s) {
    double* const W = static_cast<double*>(workspace);
    double* const dinv = W + K * kLdlP;
    const int64_t pairs = K * K / 2;
    hipLaunchKernelGGL(ldl_init_kernel, dim3(static_cast<unsigned>((pairs + 255) / 256)), dim3(256), 0, s, H, U, K,
                       info);
    if (hipGetLastError() != hipSuccess) return hipErrorLaunchFailure;
    hipLaunchKernelGGL(ldl_diag_kernel, dim3(1), dim3(256), 0, s, U, K, K - kLdlP, D, info, dinv);
    if (hipGetLastError() != hipSuccess) return hipErrorLaunchFailure;
    for (int64_t c0 = K - kLdlP; c0 > 0; c0 -= kLdlP) {
        const int64_t rows4 = c0 / 4;
        hipLaunchKernelGGL(ldl_strip_kernel, dim3(static_cast<unsigned>(rows4 < 1024 ? rows4 : 1024)), dim3(256), 0,
                           s, U, K, c0, dinv, W);
        if (hipGetLastError() != hipSuccess) return hipErrorLaunchFailure;
        const unsigned nt = static_cast<unsigned>(c0 / kLdlP);
        hipLaunchKernelGGL(ldl_trailing_kernel, dim3(nt * (nt + 1) / 2), dim3(256), 0, s, U, K, c0, W, D, info, dinv);
        if (hipGetLastError() != hipSuccess) return hipErrorLaunchFailure;
    }
    return hipSuccess;
}

}  // namespace unisvq
