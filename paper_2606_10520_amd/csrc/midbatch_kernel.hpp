// Batch product y = x * W_hat^T for 17 to 64 tokens on gfx950 (the kernel
// template; instantiated per weight format).  Internal header.
//
// A workgroup owns RB 16-row blocks over all of K; its WV wavefronts split the
// packets (two 128-column groups) round robin and meet in LDS once at the
// end, as in the small-batch kernel, so there are no partial sums in memory
// and no second launch.  Per group a wavefront holds the activation operands
// of all MT token tiles in registers (the same for its RB row blocks), decodes
// one 16 x 128 weight tile at a time on the matrix cores into its LDS tile,
// reads it back as the B operand and multiplies.  Every operand register is
// requested anew right after its last use: an activation tile for the next
// group, a packet piece for the wavefront's next packet; so the loads of the
// next step fly under the products of this one, without branches or moves.
//
// Bound: the activations that every workgroup reads (32 MT K bytes, from
// the L2) at low RB, the decode's issue slots and the products at high RB.
#pragma once

#include "common.hpp"
#include "decode.hpp"

namespace unisvq {

// Row blocks are numbered over the batch; problem i's start at rb_begin, a
// multiple of RB.
struct MidProb {
    const uint8_t* packed;   // full format, or codes only when `affine` is set
    const uint8_t* affine;   // shared affine block (codes-only format), else null
    const _Float16* x;       // fp16, row-major or tiled (bf16 activations arrive as their scaled tiled copy)
    const float* inv_scale;  // per token (scaled copies), else null
    void* y;                 // [M][N]
    int N, K, rb_begin, affine_one;
};

struct MidBatch {
    MidProb p[kMaxBatch];
    int count, M, y_dtype, tiled;
};

namespace {

constexpr int kMidRow = kGroup + 16;  // halves per decoded row of a wavefront tile (32-byte pad)
constexpr int kMidTile = 16 * kMidRow;

template <int MT, int RB, int WV>
constexpr int mid_lds_bytes() {
    constexpr int tiles = WV * kMidTile * 2, red = WV * RB * MT * 64 * 16;
    return tiles > red ? tiles : red;
}

template <int MT, int RB, int WV, bool SHARED>
__global__ __launch_bounds__(WV * 64, WV / 4) void mid_kernel(const MidBatch batch) {
    __shared__ __attribute__((aligned(16))) unsigned char lds[mid_lds_bytes<MT, RB, WV>()];
    // problem of this workgroup (uniform scalar selection)
    const int g0 = static_cast<int>(blockIdx.x) * RB;
    MidProb pb = batch.p[0];
#pragma unroll
    for (int i = 1; i < kMaxBatch; ++i)
        if (i < batch.count && g0 >= batch.p[i].rb_begin) pb = batch.p[i];
    const int M = batch.M, K = pb.K;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int groups = K >> 7;
    const int packets = (groups + 1) >> 1;
    const int rb0 = g0 - pb.rb_begin, nrb = pb.N / kRowBlock;

    constexpr uint32_t kBlockBytes = SHARED ? kCodeGroupBlockBytes : kGroupBlockBytes;
    const __amdgpu_buffer_rsrc_t rw = make_rsrc(pb.packed, static_cast<uint32_t>(nrb) * groups * kBlockBytes);
    const __amdgpu_buffer_rsrc_t ra = make_rsrc(
        pb.affine, SHARED ? static_cast<uint32_t>(pb.affine_one ? 1 : (groups + 1) / 2) * kAffineRecordBytes : 0u);
    // Tokens at or past M: past the end of a row-major buffer (they read
    // zeros), zero rows of a tiled one.  Operand of token tile i, 32-column
    // slice c of group g, lane (m = lane % 16, kb = lane / 16): token 16 i + m,
    // columns 128 g + 32 c + 8 kb .. + 7; in the tiled layout 1 KB per (tile, slice)
    // in lane order.
    const __amdgpu_buffer_rsrc_t rx =
        make_rsrc(pb.x, static_cast<uint32_t>(batch.tiled ? (M + 15) / 16 * 16 : M) * K * 2u);
    const uint32_t xlane = batch.tiled ? 16u * lane : (static_cast<uint32_t>(lane & 15) * K + 8 * (lane >> 4)) * 2u;
    const uint32_t xslice = batch.tiled ? 1024u : 64u;
    const uint32_t xtile = 32u * static_cast<uint32_t>(K);  // 16 tokens, either way
    auto load_x = [&](int g, int i, f16x8 (&xa)[4]) {
        const uint32_t base = g < groups ? xlane + static_cast<uint32_t>(g) * 4u * xslice + i * xtile : kOutOfRange;
#pragma unroll
        for (int c = 0; c < 4; ++c) xa[c] = __builtin_bit_cast(f16x8, ld128(rx, base + c * xslice));
    };
    auto load = [&](int p, int b, Piece& pc) {
        const int rb = rb0 + b;
        const uint32_t rowblk = static_cast<uint32_t>(rb) * groups * kBlockBytes;
        const int gend = rb < nrb ? groups : 0;  // (a row block that no problem has reads zeros)
        if constexpr (SHARED)
            load_packet_shared_flat<true>(rw, ra, rowblk, p, gend, pb.affine_one, lane, pc);
        else
            load_packet_flat<true>(rw, rowblk, p, gend, lane, pc);
    };

    const int j = lane & 3;
    const DecLane dl = make_dec_lane(j);
    _Float16* const wtile = reinterpret_cast<_Float16*>(lds) + wave * kMidTile;
    _Float16* const wrow = wtile + (lane >> 2) * kMidRow;
    const _Float16* const wlane = wtile + (lane & 15) * kMidRow + 8 * (lane >> 4);
    f32x4 acc[RB][MT];
#pragma unroll
    for (int b = 0; b < RB; ++b)
#pragma unroll
        for (int i = 0; i < MT; ++i) acc[b][i] = f32x4{0.f, 0.f, 0.f, 0.f};

    Piece pc[RB];
    f16x8 xa[MT][4];
#pragma unroll
    for (int b = 0; b < RB; ++b) load(wave, b, pc[b]);
#pragma unroll
    for (int i = 0; i < MT; ++i) load_x(2 * wave, i, xa[i]);
    for (int p = wave; p < packets; p += WV) {  // uniform
#pragma unroll
        for (int jj = 0; jj < 2; ++jj) {
            const int gnext = jj == 0 ? 2 * p + 1 : 2 * (p + WV);
#pragma unroll
            for (int b = 0; b < RB; ++b) {
                DecOps ops;
                prepare(pc[b], dl, jj, ops);
                f32x4 w0[4], w1[4];
                decode_half<0>(ops, w0);
                decode_half<1>(ops, w1);
#pragma unroll
                for (int n = 0; n < 4; ++n) store_w4(w0[n], wrow + 16 * n + 4 * j);
#pragma unroll
                for (int n = 0; n < 4; ++n) store_w4(w1[n], wrow + 16 * (4 + n) + 4 * j);
                if (jj == 1) load(p + WV, b, pc[b]);
                f16x8 wb[4];
#pragma unroll
                for (int c = 0; c < 4; ++c) wb[c] = *reinterpret_cast<const f16x8*>(wlane + 32 * c);
#pragma unroll
                for (int i = 0; i < MT; ++i) {
#pragma unroll
                    for (int c = 0; c < 4; ++c)
                        acc[b][i] = __builtin_amdgcn_mfma_f32_16x16x32_f16(xa[i][c], wb[c], acc[b][i], 0, 0, 0);
                    if (b == RB - 1) load_x(gnext, i, xa[i]);
                }
            }
        }
    }

    // The wavefronts meet in LDS (over the decode tiles): accumulators in lane
    // order, summed in wavefront order.  D lane layout: row lane % 16, tokens
    // 16 i + 4 (lane / 16) + e.
    __syncthreads();
    f32x4* const red = reinterpret_cast<f32x4*>(lds);  // [wave][row block][token tile][lane]
#pragma unroll
    for (int b = 0; b < RB; ++b)
#pragma unroll
        for (int i = 0; i < MT; ++i) red[((wave * RB + b) * MT + i) * 64 + lane] = acc[b][i];
    __syncthreads();
    for (int q = threadIdx.x; q < RB * MT * 64; q += WV * 64) {
        f32x4 v = red[q];
#pragma unroll
        for (int w = 1; w < WV; ++w) v += red[w * RB * MT * 64 + q];
        const int ln = q & 63, bi = q >> 6, b = bi / MT, i = bi % MT;
        if (rb0 + b >= nrb) continue;
        const int row = (rb0 + b) * kRowBlock + (ln & 15);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int t = 16 * i + 4 * (ln >> 4) + e;
            if (t < M)
                store_out(pb.y, static_cast<int64_t>(t) * pb.N + row, pb.inv_scale ? v[e] * pb.inv_scale[t] : v[e],
                          batch.y_dtype);
        }
    }
}

template <int MT, int RB, int WV, bool SHARED>
hipError_t mid_launch(const MidBatch& b, int blocks, hipStream_t s) {
    hipLaunchKernelGGL((mid_kernel<MT, RB, WV, SHARED>), dim3(static_cast<unsigned>(blocks)), dim3(WV * 64), 0, s, b);
    return hipGetLastError();
}

template <int MT, bool SHARED>
hipError_t mid_launch_rb(const MidBatch& b, int rb, int blocks, hipStream_t s) {
    switch (rb) {
        case 6: if constexpr (MT <= 3) return mid_launch<MT, 6, 8, SHARED>(b, blocks, s); return hipErrorInvalidValue;
        case 4: return mid_launch<MT, 4, 8, SHARED>(b, blocks, s);
        case 3: return mid_launch<MT, 3, 8, SHARED>(b, blocks, s);
        case 2: return mid_launch<MT, 2, 8, SHARED>(b, blocks, s);
        default: return mid_launch<MT, 1, 8, SHARED>(b, blocks, s);
    }
}

template <bool SHARED>
hipError_t mid_launch_format(const MidBatch& b, int rb, int blocks, hipStream_t s) {
    return b.M <= 32 ? mid_launch_rb<2, SHARED>(b, rb, blocks, s)
                     : (b.M <= 48 ? mid_launch_rb<3, SHARED>(b, rb, blocks, s) : mid_launch_rb<4, SHARED>(b, rb, blocks, s));
}

}  // namespace

hipError_t mid_launch_full(const MidBatch& b, int rb, int blocks, hipStream_t s);
hipError_t mid_launch_shared(const MidBatch& b, int rb, int blocks, hipStream_t s);

}  // namespace unisvq
