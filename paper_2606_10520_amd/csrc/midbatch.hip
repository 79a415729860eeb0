// Batch products for 17 to 64 tokens: the choice of a workgroup's height, the
// launch, and the full-format kernels (the codes-only ones are compiled in a
// file of their own).
#include "midbatch_kernel.hpp"

namespace unisvq {

hipError_t mid_launch_full(const MidBatch& b, int rb, int blocks, hipStream_t s) {
    return mid_launch_format<false>(b, rb, blocks, s);
}

namespace {

constexpr int kMidWaves = 8;
constexpr int kCus = 256;

// Row blocks per workgroup, and with it the rounds of workgroups over the CUs:
// the fewest rounds times the time of one, taken as 3 + rb * (packets per
// wavefront) in units of one packet's work (the fixed part is the wait for the
// first loads and the final reduction); ties go to the taller workgroup.  Within
// 3% of the best height on 40 batches (10 sets of 1024 to 57344 rows, K 1024 to
// 28672, at 17, 32, 48 and 64 tokens), e.g. 7B q+k+v, 32 tokens, heights 1 / 2 /
// 3 / 4 / 6: 19.5 / 17.9 / 22.5 / 17.4 / 21.9 us, 4 chosen.
int mid_height(const int64_t* N, int count, int64_t K, int64_t M, int64_t& rounds) {
    const int64_t units = ((K / kGroup + 1) / 2 + kMidWaves - 1) / kMidWaves;
    constexpr int kHeights[] = {6, 4, 3, 2, 1};
    int best = 1;
    int64_t best_cost = -1;
    for (const int rb : kHeights) {
        if (rb == 6 && M > 48) continue;  // (registers)
        int64_t wgs = 0;
        for (int i = 0; i < count; ++i) wgs += (N[i] / kRowBlock + rb - 1) / rb;
        const int64_t r = (wgs + kCus - 1) / kCus, cost = r * (3 + rb * units);
        if (best_cost < 0 || cost < best_cost) {
            best = rb;
            best_cost = cost;
            rounds = r;
        }
    }
    return best;
}

}  // namespace

// Against the tiled product with its K split, partial sums and second launch
// (us, this kernel against that one; rows: all problems' output rows together):
//  * fewer than 32768 rows, to 32 tokens always: 7B layer, f16, o 8.8 / 14.8 (17
//    tokens), 11.5 / 15.7 (32), q+k+v 16.6 / 25.2, gate+up 23.1 / 37.6.  (Narrow
//    and long the tiled product would win, 512 rows, K = 28672 35.1 / 18.8, but a
//    batch and each of its problems alone take one kernel here and so agree
//    bit for bit.)
//  * to 64 tokens from the rows on where reading M * K activations into every
//    workgroup is less than what the tiled product, which spreads K over the
//    chip, spends on its partial sums: rows (padded M * K - 2^18) / 128, 6144 at
//    most (f16, 64 tokens: K = 8192, 1024 rows 18.9 / 17.6, 2048 19.0 / 19.8; K =
//    14336, 4096 rows 31.1 / 26.7, 5120 35.6 / 38.4; K = 28672, 2048 rows 54.3 /
//    28.1, 6144 66.6 / 67.0, 8192 68.7 / 80.9; 7B down 25.2 / 26.0).
//  * 32768 rows and more, where the tiled product no longer splits K: to 32
//    tokens up to 49152 rows if K gives half the wavefronts a packet (K = 512,
//    32768 rows 12.5 / 11.4, K = 1024, 49152 rows 19.8 / 20.8, K = 2048 30.1 / 35.6, but 65536
//    rows 41.6 / 37.7), and any number from K = 4096 on (65536 rows 60.5 / 65.0,
//    128256 rows 113 / 118, 70B gate+up 96 / 115), from row-major activations
//    while a CU's share is below 2^19 (K = 5120, 128256 rows, 32 tokens 153 / 142).
//    Above 32 tokens not (K = 1024 21.7 / 15.8, K = 2048 28.6 / 25.9).
//  * K < 512, where neither splits K and one wavefront of eight has a packet: up
//    to 2^19 rows * padded tokens (K = 256, 32 tokens: 16384 rows 6.9 / 8.3, 28672
//    rows 11.6 / 9.0, 65536 rows 22.5 / 11.4; 64 tokens: 10240 rows 8.1 / 8.1).
// Every workgroup reads all activations, row-major ones in pieces of 64 bytes at
// 15 bytes a clock and CU, the tiled layout at more than twice that.  So f16
// activations are copied into it (a launch of 2 us: K = 256 5.8 -> 7.8 us) from a
// share of rounds * M * K of 2^17 on (2^18 up to 32 tokens): copied against
// row-major, 64 tokens: K = 2048, 1024 rows 8.6 / 11.4, o 12.7 / 19.7, q+k+v 21.4 /
// 25.3, gate+up 33.6 / 44.8; 24 tokens: K = 11008 17.4 / 21.3, but K = 8192 (a
// share of 3 * 2^16) 23.7 / 21.1.  Above 32 tokens a larger share without room for
// the copy goes to the tiled product, and a smaller one needs its rows too (K =
// 2048, 64 rows, 56 tokens 10.2 / 9.4).
MidPlan mid_plan(const int64_t* N, int count, int64_t K, int64_t M, bool bf16, bool room) {
    if (M <= kSkinnyMaxM || M > kMidMaxM) return {false, false};
    if ((M + 15) / 16 * 16 * K * 2 > kMaxBufferBytes) return {false, false};  // (32-bit offsets: the tiled product slices)
    int64_t rows = 0, rounds = 1;
    for (int i = 0; i < count; ++i) rows += N[i];
    mid_height(N, count, K, M, rounds);
    const int64_t padded = M <= 32 ? 32 : (M + 15) / 16 * 16;
    const int64_t share = rounds * M * K;
    const bool copy = bf16 || (room && share >= (M <= 32 ? 1 << 18 : 1 << 17));
    bool serves;
    if (K < 512) {
        serves = rows * padded <= 1 << 19;
    } else if (M <= 32) {
        serves = rows < 32768 || (K >= 1024 && rows <= 49152) || (K >= 4096 && (copy || share < 1 << 19));
    } else {
        const int64_t need = (padded * K - (copy ? 1 << 18 : 1 << 16)) / 128;
        serves = rows < 32768 && (copy || share < 1 << 17) && rows >= (need < 6144 ? need : 6144);
    }
    return {serves, copy};
}

hipError_t launch_mid_batch(const SkinnyProblem* probs, int count, int64_t M, bool tiled, int y_dtype, hipStream_t s) {
    if (count < 1 || count > kMaxBatch || M < 1 || M > kMidMaxM) return hipErrorInvalidValue;
    int64_t ns[kMaxBatch], kmax = 0, rounds = 0;
    for (int i = 0; i < count; ++i) {
        ns[i] = probs[i].N;
        kmax = probs[i].K > kmax ? probs[i].K : kmax;
    }
    const int rb = mid_height(ns, count, kmax, M, rounds);
    MidBatch b{};
    int64_t start = 0;
    for (int i = 0; i < count; ++i) {
        const SkinnyProblem& q = probs[i];
        b.p[i] = MidProb{q.packed, q.affine, q.x, q.inv_scale, q.y, static_cast<int>(q.N), static_cast<int>(q.K),
                         static_cast<int>(start), q.affine_one};
        start += (q.N / kRowBlock + rb - 1) / rb * rb;
    }
    b.count = count;
    b.M = static_cast<int>(M);
    b.y_dtype = y_dtype;
    b.tiled = tiled;
    const int blocks = static_cast<int>(start / rb);
    return probs[0].affine ? mid_launch_shared(b, rb, blocks, s) : mid_launch_full(b, rb, blocks, s);
}

}  // namespace unisvq
