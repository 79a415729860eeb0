// LDLQ on gfx950: nearest-codeword rounding with Hessian error feedback
// (Sec. 3.2.2, Eq. 7).  Vectors of 4 columns are rounded left to right; the
// target of vector j is u = W_j + sum_{k < 4j} E_k U[k][j] (E = W - W_hat,
// U the unit upper block-triangular factor of H = U D U^T).
//
// The running feedback F[r][c] = sum_k E[r][k] U[k][c] lives in the
// workspace (fp64).  Every F element is one fma chain in increasing k, exactly
// the sum of the definition, and the decision on u = W + F is taken on fp64
// distances with the nearest-codeword quantiser's operation order and tie
// rule: the codes equal a plain sequential evaluation of Eq. 7 bit for bit.
//
// Columns go in blocks of 128 (one group), one launch per block b with two
// kinds of workgroups:
//  * step: 16 rows; adds block b - 1's errors to block b, rounds the block's
//    32 vectors and leaves the errors E_b in the workspace where F's block b
//    was (nothing reads that again);
//  * far: F += (E_{b-2}, E_{b-1}) U for the column blocks b + 1, b + 3, ...,
//    a rank-256 update, so that F is read and written half as often as with
//    one update per block.  Block c thus has E_0 .. E_{c-2} when its step
//    comes and the step adds E_{c-1} itself; the far workgroups write only
//    blocks that no step of the launch reads.
// The rounding is a serial chain of 32 vectors on one wavefront per SIMD;
// the far products fill the matrix cores beside it.
//
// All products run on v_mfma_f64_16x16x4f64, which rounds like four fmas in
// increasing k (compared with host fma chains over 76800 sums, subnormal
// products among them: equal bit for bit).  Lanes: A[i][k] at lane i + 16 k,
// B[k][j] at lane j + 16 k, result D[i][j] at lane j + 16 (i % 4), item i / 4.
//
// Workspace: per (16-row block, column block) 2048 doubles, as F eight
// 16 x 16 tiles in result order ([tile][lane][item]), tile 4 h + q holding
// columns 64 h + 4 j + q (so that a lane holds whole vectors and reads 16 and
// 32 contiguous bytes of a row of U), as E 32 steps of 4 columns in operand
// order ([step / 2][lane][step % 2]).
//
// 4096 x 4096, MI355X: 2.05 ms in 32 launches, 4.2 ms in 64 before (step 64 us a
// block with 256 fp64 distances per vector spread over a wavefront per row,
// update 82 us with fp64 vector fmas and rank 128).  A step alone takes 24 us
// (5 of them loads, tables and the product inside the block); with all its far
// workgroups a launch takes 97 us, about the step's time plus that of the
// matrix instructions (51 us at their rate): fp64 matrix and vector
// instructions share their unit, so the two overlap little.
#include <utility>

#include "common.hpp"

namespace unisvq {
namespace {

constexpr int kLdlqBlock = 128;          // columns per block (= one group)
constexpr int kBlkDoubles = 16 * kLdlqBlock;  // workspace doubles per (16 rows, block)
constexpr int kHalf = 64;                // columns rounded between two products inside a block
constexpr int kFarRows = 128;            // far workgroup: 128 rows x 64 columns, 32 x 64 per wavefront
constexpr int kFarCols = 64;
typedef double f64x2 __attribute__((ext_vector_type(2)));
typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef f64x4 f64x4m __attribute__((aligned(16)));  // in the workspace, which is 16-byte aligned

__device__ inline double h2d(uint16_t h) {
    return static_cast<double>(static_cast<float>(__builtin_bit_cast(_Float16, h)));
}

// Value of lane L of each row of 16 lanes.
template <int L>
__device__ inline float row_bcast(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0x150 + L, 0xf, 0xf, true));
}
// Value of lane K of each quad.
template <int K>
__device__ inline double quad_bcast(double v) {
    const uint2 w = __builtin_bit_cast(uint2, v);
    return __builtin_bit_cast(double, uint2{static_cast<uint32_t>(__builtin_amdgcn_mov_dpp(static_cast<int>(w.x), 0x55 * K, 0xf, 0xf, true)),
                                            static_cast<uint32_t>(__builtin_amdgcn_mov_dpp(static_cast<int>(w.y), 0x55 * K, 0xf, 0xf, true))});
}
// Rotation by R inside each row of 16 lanes.
template <int R>
__device__ inline int row_ror(int v) {
    return __builtin_amdgcn_mov_dpp(v, 0x120 + R, 0xf, 0xf, true);
}
template <int R>
__device__ inline float row_ror(float v) {
    return __builtin_bit_cast(float, row_ror<R>(__builtin_bit_cast(int, v)));
}
template <int R>
__device__ inline double row_ror(double v) {
    const uint2 w = __builtin_bit_cast(uint2, v);
    return __builtin_bit_cast(double, uint2{static_cast<uint32_t>(row_ror<R>(static_cast<int>(w.x))),
                                            static_cast<uint32_t>(row_ror<R>(static_cast<int>(w.y)))});
}

// Squared distance from u to codeword c, accumulated with fmas in component order.
__device__ inline double cw_dist(const double (&c)[4], const double (&u)[4]) {
    double d = 0.0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const double e = c[k] - u[k];
        d = __builtin_fma(e, e, d);
    }
    return d;
}

template <int R>
__device__ inline void min_step(double& bd, int& bi) {
    const double od = row_ror<R>(bd);
    const int oi = row_ror<R>(bi);
    if (od < bd || (od == bd && oi < bi)) {
        bd = od;
        bi = oi;
    }
}

// Squared distance from u to codeword idx (q_b = bits 2b, 2b+1) of the pair ab
// (A row-major, then B), in the quantiser's operation order (the codeword is
// exact whatever the order).
__device__ inline double cw_exact(const double* ab, int idx, const double (&u)[4]) {
    const double q0 = static_cast<double>(idx & 3), q1 = static_cast<double>((idx >> 2) & 3);
    const double q2 = static_cast<double>((idx >> 4) & 3), q3 = static_cast<double>((idx >> 6) & 3);
    double c[4];
#pragma unroll
    for (int k = 0; k < 4; ++k)
        c[k] = ab[16 + k] + ab[4 * k] * q0 + ab[4 * k + 1] * q1 + ab[4 * k + 2] * q2 + ab[4 * k + 3] * q3;
    return cw_dist(c, u);
}

// The nearest of codewords i0 <= i1 of every lane of a row of 16 lanes (the
// lowest index on equal distances), the same result in all of them; a lane
// without a candidate passes d = infinity.
__device__ inline int nearest_of_row(double d0, int i0, double d1, int i1) {
    if (d1 < d0 || (d1 == d0 && i1 < i0)) {
        d0 = d1;
        i0 = i1;
    }
    min_step<8>(d0, i0);
    min_step<4>(d0, i0);
    min_step<2>(d0, i0);
    min_step<1>(d0, i0);
    return __builtin_amdgcn_mov_dpp(i0, 0x150, 0xf, 0xf, true);  // one value per row also where NaNs made them differ
}

// All 256 codewords, sixteen per lane (q0, q1 from jl).
__device__ inline int nearest_exact(const double* ab, const double (&u)[4], int jl) {
    double bd = 0.0;
    int bi = jl;
#pragma clang loop unroll(disable)
    for (int j = 0; j < 16; ++j) {
        const double d = cw_exact(ab, jl + 16 * j, u);
        if (j == 0 || d < bd) {
            bd = d;
            bi = jl + 16 * j;
        }
    }
    return nearest_of_row(bd, bi, bd, bi);
}

// One row's search state: the row's 16 lanes share the row; lane jl.
//
// Codeword(i, j) = b' + p_i + r_j with p_i = A_0 q0' + A_1 q1' (i = q0 + 4 q1),
// r_j = A_2 q2' + A_3 q3' (j = q2 + 4 q3), q' = q - 3/2 and b' = b + 3/2 sum_k
// A_k (all exact in fp64; centred, so that the terms are small).  With t =
// u - b' its squared distance to u, less |t|^2, is
//     s_ij = (|p_i|^2 - 2 p_i t) + (|r_j|^2 - 2 r_j t) + 2 p_i r_j,
// one addition per codeword once the two 16-entry terms are there (lane i
// holds 2 p_i r_j for all j, and takes the r terms from the lanes of its
// row).  This is done in fp32 and only names the codewords that can be
// nearest: with P >= |p_i|, |r_j| and T >= |t| the sum of the roundings is
// below 63 P (P + T) 2^-24 (terms of at most P^2 + 2 P T with six roundings
// each, three bits of the index kept in the low bits of a value of at most
// 3 P^2 + 2 P T, and the last additions), so every codeword within
// 128 P (P + T) 2^-24 of the smallest is a candidate.  One candidate: it is
// the nearest (the fp64 distances round by at most 2^-50 (P + T)^2, less than
// the slack up to T = 2^28 P).  Several: their fp64 distances decide, at most
// two per lane (both named by the search).  More in a lane, or T / P or a
// value beyond these ranges: all 256.  (Several candidates
// come up in about one vector of 1000 on a wavefront of four rows, but the
// slowest of 1024 wavefronts sets the launch's end: with all 256 each time, at
// one vector of 140, this path took 10 of a block's 26 us.)
struct RowSearch {
    float pm[4], rm[4];  // -2 p_i, -2 r_i of lane i
    float pn, rn;        // |p_i|^2, |r_i|^2
    float g[16];         // 2 p_i r_j
    float tolc;          // P 2^-17
    float tolmax;        // the tolerance at T = 2^28 P
};

__device__ inline void build_search(const double* ab, int jl, RowSearch& s) {
    const double q0 = static_cast<double>(jl & 3) - 1.5, q1 = static_cast<double>(jl >> 2) - 1.5;
    double pn = 0.0, rn = 0.0, d2 = 0.0, d3 = 0.0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const double a2 = ab[4 * k + 2], a3 = ab[4 * k + 3];
        const double p = ab[4 * k] * q0 + ab[4 * k + 1] * q1;
        const double r = a2 * q0 + a3 * q1;
        s.pm[k] = static_cast<float>(-2.0 * p);
        s.rm[k] = static_cast<float>(-2.0 * r);
        pn += p * p;
        rn += r * r;
        d2 += 2.0 * p * a2;
        d3 += 2.0 * p * a3;
    }
    s.pn = static_cast<float>(pn);
    s.rn = static_cast<float>(rn);
#pragma unroll
    for (int j = 0; j < 16; ++j)
        s.g[j] = static_cast<float>(d2 * ((j & 3) - 1.5) + d3 * ((j >> 2) - 1.5));
    float m = fmaxf(s.pn, s.rn);
    m = fmaxf(m, row_ror<8>(m));
    m = fmaxf(m, row_ror<4>(m));
    m = fmaxf(m, row_ror<2>(m));
    m = fmaxf(m, row_ror<1>(m));
    s.tolc = sqrtf(m) * (1.001f / 131072.0f);
    s.tolmax = fminf(m * 2048.0f, 1e25f);
}

// The minimum as one instruction (fminf first quiets both operands: sixteen
// more per vector).  Its result must not go straight into a lane exchange:
// the compiler does not see that a vector instruction wrote it.
__device__ inline float min_f(float a, float b) {
    float r;
    asm("v_min_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

// x_j = g[j] + (r term of lane j), j % 8 in its low three bits.
template <int J>
__device__ inline float tagged(const RowSearch& s, float beta) {
    const uint32_t x = __builtin_bit_cast(uint32_t, s.g[J] + row_bcast<J>(beta));
    return __builtin_bit_cast(float, (x & ~7u) | static_cast<uint32_t>(J & 7));
}
// The two smallest of a chain (a value below both moves the smaller one up).
template <int J>
__device__ inline void scan(const RowSearch& s, float beta, float& m1, float& m2) {
    const float xi = tagged<J>(s, beta);
    m2 = __builtin_amdgcn_fmed3f(m1, m2, xi);
    m1 = min_f(m1, xi);
}
template <int... J>
__device__ inline void scan_all(const RowSearch& s, float beta, float& a1, float& a2, float& b1, float& b2,
                                std::integer_sequence<int, J...>) {
    ((scan<J>(s, beta, a1, a2), scan<J + 8>(s, beta, b1, b2)), ...);
}

// Number of values x_j of this lane that pass the threshold.
template <int... J>
__device__ inline void count_all(const RowSearch& s, float beta, float alpha, float thr, int& n,
                                 std::integer_sequence<int, J...>) {
    ((n += tagged<J>(s, beta) + alpha <= thr), ...);
}

// j of the tagged value m, the smaller of chain a's (a1, j < 8) and chain b's.
__device__ inline int chain_index(float m, float a1) {
    return static_cast<int>(__builtin_bit_cast(uint32_t, m) & 7u) + (m == a1 ? 0 : 8);
}

// What a wavefront of a step workgroup keeps: four rows (lane / 16), lane jl
// of a row owns vector jl of the current half block (f, w: its four columns).
struct StepState {
    RowSearch s;
    const double* ab;  // the row's pair
    double f[4], b[4];  // b: the centre b'
    float4 w;
    double arow[4], brow;   // row jl % 4 of A and B: the component that the lane subtracts
    uint32_t code;          // index chosen for the lane's own vector
    int jl;
};

// The value of lane `from` / 4 (a byte address, as the exchange takes it).
__device__ inline float lane_get(int from, float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute(from, __builtin_bit_cast(int, v)));
}
__device__ inline double lane_get(int from, double v) {
    const uint2 w = __builtin_bit_cast(uint2, v);
    return __builtin_bit_cast(double, uint2{static_cast<uint32_t>(__builtin_amdgcn_ds_bpermute(from, static_cast<int>(w.x))),
                                            static_cast<uint32_t>(__builtin_amdgcn_ds_bpermute(from, static_cast<int>(w.y)))});
}

// Vector v of the half block.  (A loop with exchanges through the LDS unit, not
// sixteen copies with the lane fixed in each: those and their rare paths
// outgrew the instruction cache.)
__device__ inline void step_vector(StepState& st, int v, const f64x2* us, const float* wrow, double* es) {
    const int from = 4 * ((threadIdx.x & 48) + v);
    // target of the lane's own vector (only lane v's is final)
    const double u[4] = {static_cast<double>(st.w.x) + st.f[0], static_cast<double>(st.w.y) + st.f[1],
                         static_cast<double>(st.w.z) + st.f[2], static_cast<double>(st.w.w) + st.f[3]};
    float t[4], tn = 0.0f;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        t[k] = static_cast<float>(u[k] - st.b[k]);
        tn += fabsf(t[k]);
    }
    float tol = fmaf(131072.0f, st.s.tolc, tn) * st.s.tolc;
    float tb[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) tb[k] = lane_get(from, t[k]);
    tol = lane_get(from, tol);
    __builtin_amdgcn_sched_barrier(0);
    // U's rows of the vector and its weight, read after the exchange (the LDS unit
    // answers in order) so that they land under the search
    f64x2 uk[4][2];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        uk[k][0] = us[((4 * v + k) * 2) * 16];
        uk[k][1] = us[((4 * v + k) * 2 + 1) * 16];
    }
    const float wv = wrow[4 * v];
    __builtin_amdgcn_sched_barrier(0);
    float al = st.s.pn, be = st.s.rn;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        al = fmaf(st.s.pm[k], tb[k], al);
        be = fmaf(st.s.rm[k], tb[k], be);
    }
    const bool range = tol > 1e-25f && tol < st.s.tolmax;  // (false for NaN)
    // two chains of eight (a1 <= a2, b1 <= b2), then the two smallest of both
    float a1 = __builtin_inff(), a2 = a1, b1 = a1, b2 = a1;
    scan_all(st.s, be, a1, a2, b1, b2, std::make_integer_sequence<int, 8>());
    const float m1 = min_f(a1, b1), am = __builtin_amdgcn_fmed3f(a1, b1, __builtin_inff());
    const float m2 = min_f(am, min_f(a2, b2));
    const float y1 = m1 + al, y2 = m2 + al;
    float m = y1;
    m = fminf(m, row_ror<8>(m));
    m = fminf(m, row_ror<4>(m));
    m = fminf(m, row_ror<2>(m));
    m = fminf(m, row_ror<1>(m));
    const float thr = m + tol;
    const bool win = y1 <= thr;
    // one candidate in each of the four rows, all in range
    const bool clear = __popcll(__ballot(win)) == 4 && __ballot(y2 <= thr || !range) == 0;
    int idx;
    if (clear) {  // uniform
        // (a1 and b1 are not equal here: both would have passed)
        idx = win ? st.jl + 16 * chain_index(m1, a1) : 0;
        idx |= row_ror<8>(idx);
        idx |= row_ror<4>(idx);
        idx |= row_ror<2>(idx);
        idx |= row_ror<1>(idx);
    } else {
        double ub[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) ub[k] = lane_get(from, u[k]);
        int n = 0;  // this lane's candidates
        count_all(st.s, be, al, thr, n, std::make_integer_sequence<int, 16>());
        if (__ballot(n > 2 || !range) == 0) {
            // the two smallest: m1 of chain a or b, m2 the other's first or the same's second
            const bool a_first = a1 <= b1;
            const float x1 = a_first ? a1 : b1;
            const int i1 = st.jl + 16 * static_cast<int>((__builtin_bit_cast(uint32_t, x1) & 7u) + (a_first ? 0u : 8u));
            const bool other = (a_first ? b1 : a1) <= (a_first ? a2 : b2);  // m2 comes from the other chain
            const float x2 = other ? (a_first ? b1 : a1) : (a_first ? a2 : b2);
            const int i2 = st.jl + 16 * static_cast<int>((__builtin_bit_cast(uint32_t, x2) & 7u) + (a_first != other ? 0u : 8u));
            const double d1 = cw_exact(st.ab, i1, ub), d2 = cw_exact(st.ab, i2, ub);
            idx = nearest_of_row(win ? d1 : __builtin_inf(), i1, y2 <= thr ? d2 : __builtin_inf(), i2);
        } else {
            idx = nearest_exact(st.ab, ub, st.jl);
        }
    }
    if (st.jl == v) st.code = static_cast<uint32_t>(idx);
    // error of component jl % 4 (the codeword is exact), then all four
    double c = st.brow;
#pragma unroll
    for (int k = 0; k < 4; ++k) c = c + st.arow[k] * static_cast<double>((idx >> (2 * k)) & 3);
    const double e = static_cast<double>(wv) - c;
    es[64 * v] = e;  // (four lanes hold the same component: the same value)
    const double ev[4] = {quad_bcast<0>(e), quad_bcast<1>(e), quad_bcast<2>(e), quad_bcast<3>(e)};
    // feed the errors forward, in increasing k, to the half block's columns
    // (vectors up to v get values that are not read again)
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        st.f[0] = __builtin_fma(ev[k], uk[k][0].x, st.f[0]);
        st.f[1] = __builtin_fma(ev[k], uk[k][0].y, st.f[1]);
        st.f[2] = __builtin_fma(ev[k], uk[k][1].x, st.f[2]);
        st.f[3] = __builtin_fma(ev[k], uk[k][1].y, st.f[3]);
    }
}
// Step workgroup: rows 16 rb .. 16 rb + 15 of block b.  LDS: U's 64 x 64
// diagonal block of the current half (two f64x2 per vector and row, split so
// that sixteen lanes read 256 contiguous bytes), F in result order, E in
// operand order per half, the weights.
struct StepLds {
    f64x2 us[kHalf * 2 * 16];
    double fs[8 * 4 * 64];
    double es[2][16 * 64];
    float ws[16][kLdlqBlock + 4];
    double ab[16][20];  // the rows' pairs: A row-major, then B
};

__device__ inline void ldlq_step(StepLds& sh, int64_t K, int b, int64_t rb, const float* __restrict__ W,
                                 const double* __restrict__ U, const uint16_t* __restrict__ A,
                                 const uint16_t* __restrict__ B, int64_t affine_groups, double* F,
                                 uint8_t* __restrict__ codes) {
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int jl = lane & 15, lk = lane >> 4;
    const int64_t groups = K / kLdlqBlock;
    double* const blk = F + (rb * groups + b) * kBlkDoubles;
    const double* const Ud = U + static_cast<int64_t>(b) * kLdlqBlock * (K + 1);  // the block's diagonal part
    const int64_t row = 16 * rb + 4 * wave + lk;  // this lane's row of the rounding

    // weights and U's first diagonal half block to LDS
    {
        const float* wp = W + (16 * rb + (t >> 4)) * K + static_cast<int64_t>(b) * kLdlqBlock + 8 * (t & 15);
        const float4 w0 = *reinterpret_cast<const float4*>(wp), w1 = *reinterpret_cast<const float4*>(wp + 4);
        f64x2 v[8];
#pragma unroll
        for (int n = 0; n < 8; ++n) {
            const int i = t + 256 * n, r = i >> 5, c2 = i & 31;
            v[n] = *reinterpret_cast<const f64x2*>(Ud + static_cast<int64_t>(r) * K + 2 * c2);
        }
        // (thread t: element t % 16 of A and, for four of them, t % 4 of B, row t / 16)
        const int64_t ar = 16 * rb + (t >> 4);
        const int64_t set = affine_groups == 0 ? ar * groups + b : (affine_groups == 1 ? 0 : b);
        const uint16_t av = A[set * 16 + (t & 15)], bv = B[set * 4 + (t & 3)];
        sh.ab[t >> 4][t & 15] = h2d(av);
        sh.ab[t >> 4][16 + (t & 3)] = h2d(bv);
        *reinterpret_cast<float4*>(&sh.ws[t >> 4][8 * (t & 15)]) = w0;
        *reinterpret_cast<float4*>(&sh.ws[t >> 4][8 * (t & 15) + 4]) = w1;
#pragma unroll
        for (int n = 0; n < 8; ++n) {
            const int i = t + 256 * n, r = i >> 5, c2 = i & 31;
            sh.us[(2 * r + (c2 & 1)) * 16 + (c2 >> 1)] = v[n];
        }
    }
    // F of the block: this wavefront's tiles 2 wave, 2 wave + 1 (columns
    // 64 h + 4 j + q, q = q0, q0 + 1), plus the errors of block b - 1
    {
        const int h = wave >> 1, q0 = 2 * (wave & 1);
        f64x4 acc[2] = {};
        if (b >= 2) {
#pragma unroll
            for (int q = 0; q < 2; ++q)
                acc[q] = *reinterpret_cast<const f64x4m*>(blk + (4 * h + q0 + q) * 256 + 4 * lane);
        }
        if (b >= 1) {
            const double* ep = blk - kBlkDoubles + 2 * lane;
            const double* up = U + (static_cast<int64_t>(b - 1) * kLdlqBlock + lk) * K +
                               static_cast<int64_t>(b) * kLdlqBlock + kHalf * h + 4 * jl + q0;
            f64x2 ea[2][4], ub[2][4][2];
            auto fetch = [&](int ch, int buf) {
#pragma unroll
                for (int p = 0; p < 4; ++p) {
                    const int sp = 4 * ch + p;
                    ea[buf][p] = *reinterpret_cast<const f64x2*>(ep + 128 * sp);
                    ub[buf][p][0] = *reinterpret_cast<const f64x2*>(up + static_cast<int64_t>(8 * sp) * K);
                    ub[buf][p][1] = *reinterpret_cast<const f64x2*>(up + static_cast<int64_t>(8 * sp + 4) * K);
                }
            };
            fetch(0, 0);
#pragma unroll
            for (int ch = 0; ch < 4; ++ch) {
                if (ch + 1 < 4) fetch(ch + 1, (ch + 1) & 1);
#pragma unroll
                for (int p = 0; p < 4; ++p) {
                    const f64x2 e = ea[ch & 1][p], u0 = ub[ch & 1][p][0], u1 = ub[ch & 1][p][1];
                    acc[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(e.x, u0.x, acc[0], 0, 0, 0);
                    acc[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(e.x, u0.y, acc[1], 0, 0, 0);
                    acc[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(e.y, u1.x, acc[0], 0, 0, 0);
                    acc[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(e.y, u1.y, acc[1], 0, 0, 0);
                }
            }
        }
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int v = 0; v < 4; ++v) sh.fs[((4 * h + q0 + q) * 4 + v) * 64 + lane] = acc[q][v];
    }
    StepState st;
    st.ab = sh.ab[4 * wave + lk];
    st.jl = jl;
    __syncthreads();
    build_search(st.ab, jl, st.s);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        st.b[k] = st.ab[16 + k] + 1.5 * (st.ab[4 * k] + st.ab[4 * k + 1] + st.ab[4 * k + 2] + st.ab[4 * k + 3]);
        st.arow[k] = st.ab[4 * (jl & 3) + k];
    }
    st.brow = st.ab[16 + (jl & 3)];
#pragma clang loop unroll(disable)
    for (int h = 0; h < 2; ++h) {
        // (row i = lk + 4 wave of a tile is item `wave` of lane jl + 16 lk)
#pragma unroll
        for (int q = 0; q < 4; ++q) st.f[q] = sh.fs[((4 * h + q) * 4 + wave) * 64 + lane];
        st.w = *reinterpret_cast<const float4*>(&sh.ws[4 * wave + lk][kHalf * h + 4 * jl]);
        st.code = 0;
#pragma clang loop unroll(disable)
        for (int v = 0; v < kHalf / 4; ++v)
            step_vector(st, v, sh.us + jl, &sh.ws[4 * wave + lk][kHalf * h + (jl & 3)],
                        &sh.es[h][lk + 4 * wave + 16 * (jl & 3)]);
        *reinterpret_cast<uint32_t*>(codes + row * K + static_cast<int64_t>(b) * kLdlqBlock + kHalf * h + 4 * jl) =
            (st.code & 3u) | ((st.code & 12u) << 6) | ((st.code & 48u) << 12) | ((st.code & 192u) << 18);
        if (h == 0) {
            // for the second half: U's diagonal half block, and the first half's
            // rows of U for tile 4 + wave (held over the first half they spilled)
            double ub[16];
            f64x2 un[8];
            const double* up = Ud + static_cast<int64_t>(lk) * K + kHalf + 4 * jl + wave;
#pragma unroll
            for (int s = 0; s < 16; ++s) ub[s] = up[static_cast<int64_t>(4 * s) * K];
            const double* u1 = Ud + static_cast<int64_t>(kHalf) * (K + 1);
#pragma unroll
            for (int n = 0; n < 8; ++n) {
                const int i = t + 256 * n, r = i >> 5, c2 = i & 31;
                un[n] = *reinterpret_cast<const f64x2*>(u1 + static_cast<int64_t>(r) * K + 2 * c2);
            }
            __syncthreads();  // E of the half is whole, its U block is free
#pragma unroll
            for (int n = 0; n < 8; ++n) {
                const int i = t + 256 * n, r = i >> 5, c2 = i & 31;
                sh.us[(2 * r + (c2 & 1)) * 16 + (c2 >> 1)] = un[n];
            }
            f64x4 acc;
            double* const fp = sh.fs + (4 + wave) * 256 + lane;
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[i] = fp[64 * i];
#pragma unroll
            for (int s = 0; s < 16; ++s)
                acc = __builtin_amdgcn_mfma_f64_16x16x4f64(sh.es[0][64 * s + lane], ub[s], acc, 0, 0, 0);
#pragma unroll
            for (int i = 0; i < 4; ++i) fp[64 * i] = acc[i];
            __syncthreads();
        }
    }
    __syncthreads();
    // E in operand order, two steps per 16-byte piece
#pragma unroll
    for (int n = 0; n < 4; ++n) {
        const int i = t + 256 * n, sp = i >> 6;  // step pair, lane `lane`
        const double* const e = &sh.es[0][0] + 128 * sp + lane;
        *reinterpret_cast<f64x2*>(blk + 2 * i) = f64x2{e[0], e[64]};
    }
}

// Far wavefront: rows of 16-row blocks rb0, rb0 + 1, columns 64 cg .. 64 cg +
// 63: F += E U over the blocks kb0 .. b - 1 (one or two), two steps of four
// k per turn, three turns' operands in flight (with one the wavefront waited for
// its loads: a rank-256 tile took 40 us for 14 us of matrix instructions).
struct FarOps {
    f64x2 a[2];     // [row block]: steps 2 sp, 2 sp + 1
    f64x2 u[2][2];  // [step][columns q = 0, 1 / 2, 3]
};

__device__ inline void ldlq_far(int64_t N, int64_t K, int b, int64_t rb0, int64_t cg, const double* __restrict__ U,
                                double* F) {
    const int64_t rbs = N / 16;
    if (rb0 >= rbs) return;  // uniform
    const int lane = threadIdx.x & 63, jl = lane & 15, lk = lane >> 4;
    const int64_t groups = K / kLdlqBlock;
    const int64_t rb1 = rb0 + 1 < rbs ? rb0 + 1 : rb0;  // (an odd last row block is computed twice, the same values)
    const int kb0 = b >= 2 ? b - 2 : 0;
    const int turns = 16 * (b - kb0);
    const int64_t c = cg >> 1;
    const int h = static_cast<int>(cg & 1);
    double* const f0 = F + (rb0 * groups + c) * kBlkDoubles + h * 1024 + 4 * lane;
    double* const f1 = F + (rb1 * groups + c) * kBlkDoubles + h * 1024 + 4 * lane;
    const double* const e0 = F + (rb0 * groups + kb0) * kBlkDoubles + 2 * lane;
    const double* const e1 = F + (rb1 * groups + kb0) * kBlkDoubles + 2 * lane;
    const double* const up = U + (static_cast<int64_t>(kb0) * kLdlqBlock + lk) * K + cg * kFarCols + 4 * jl;
    auto fetch = [&](int sp, FarOps& o) {
        o.a[0] = *reinterpret_cast<const f64x2*>(e0 + 128 * sp);
        o.a[1] = *reinterpret_cast<const f64x2*>(e1 + 128 * sp);
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int q = 0; q < 2; ++q)
                o.u[s][q] = *reinterpret_cast<const f64x2*>(up + static_cast<int64_t>(8 * sp + 4 * s) * K + 2 * q);
    };
    f64x4 acc[2][4];
    auto mul = [&](const FarOps& o) {
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int r = 0; r < 2; ++r)
                    acc[r][q] = __builtin_amdgcn_mfma_f64_16x16x4f64(s ? o.a[r].y : o.a[r].x,
                                                                     q & 1 ? o.u[s][q >> 1].y : o.u[s][q >> 1].x,
                                                                     acc[r][q], 0, 0, 0);
    };
    FarOps o[4];
#pragma unroll
    for (int i = 0; i < 3; ++i) fetch(i, o[i]);
    const bool first = kb0 == 0;  // the first errors that this column block gets: F starts at zero
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const f64x4 v0 = *reinterpret_cast<const f64x4m*>(f0 + 256 * q), v1 = *reinterpret_cast<const f64x4m*>(f1 + 256 * q);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            acc[0][q][i] = first ? 0.0 : v0[i];
            acc[1][q][i] = first ? 0.0 : v1[i];
        }
    }
#pragma clang loop unroll(disable)
    for (int sp = 0; sp < turns; sp += 4) {  // turns is 16 or 32
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int next = sp + i + 3;
            fetch(next < turns ? next : 0, o[(i + 3) & 3]);
            mul(o[i]);
        }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        *reinterpret_cast<f64x4m*>(f0 + 256 * q) = acc[0][q];
        *reinterpret_cast<f64x4m*>(f1 + 256 * q) = acc[1][q];
    }
}

// Launch b: N / 16 step workgroups first, then the far ones (row tiles
// fastest: each XCD keeps the errors of its row tiles in its L2 for every
// column tile).  Two workgroups per CU (74 KB of LDS each).
__global__ __launch_bounds__(256, 2) void ldlq_kernel(int64_t N, int64_t K, int b, const float* __restrict__ W,
                                                      const double* __restrict__ U, const uint16_t* __restrict__ A,
                                                      const uint16_t* __restrict__ B, int64_t affine_groups,
                                                      double* F, uint8_t* __restrict__ codes) {
    __shared__ StepLds sh;
    const int64_t steps = N / 16;
    if (blockIdx.x < steps) {
        ldlq_step(sh, K, b, blockIdx.x, W, U, A, B, affine_groups, F, codes);
        return;
    }
    const int64_t id = blockIdx.x - steps, row_tiles = (N + kFarRows - 1) / kFarRows;
    const int64_t rt = id % row_tiles, ct = id / row_tiles;
    // column tile ct: half ct % 2 of block b + 1 + 2 (ct / 2)
    const int64_t cg = 2 * (b + 1 + 2 * (ct >> 1)) + (ct & 1);
    ldlq_far(N, K, b, rt * (kFarRows / 16) + 2 * __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), cg, U, F);
}

}  // namespace

// F and E share one N x K area.  The N x 128 doubles beyond it are not touched:
// they are part of the size that the interface has stated since E had an area
// of its own, and a buffer without them stays refused.
size_t ldlq_workspace_bytes(int64_t N, int64_t K) {
    return static_cast<size_t>(N) * static_cast<size_t>(K) * 8 + static_cast<size_t>(N) * kLdlqBlock * 8;
}

hipError_t launch_ldlq(int64_t N, int64_t K, const float* W, const double* U, const uint16_t* A, const uint16_t* B,
                       int64_t affine_groups, uint8_t* codes, void* workspace, hipStream_t s) {
    double* F = static_cast<double*>(workspace);
    const int blocks = static_cast<int>(K / kLdlqBlock);
    const int64_t row_tiles = (N + kFarRows - 1) / kFarRows;
    for (int b = 0; b < blocks; ++b) {
        const int64_t far = b >= 1 ? (blocks - b) / 2 : 0;  // blocks b + 1, b + 3, ...
        const int64_t grid = N / 16 + 2 * far * row_tiles;
        hipLaunchKernelGGL(ldlq_kernel, dim3(static_cast<unsigned>(grid)), dim3(256), 0, s, N, K, b, W, U, A, B,
                           affine_groups, F, codes);
        if (hipGetLastError() != hipSuccess) return hipErrorLaunchFailure;
    }
    return hipSuccess;
}

}  // namespace unisvq
