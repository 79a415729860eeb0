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
// 5% of the best height on 30 batches (K 1024 to 28672, 1024 to 57344 rows, 17
// to 64 tokens), e.g. 7B q+k+v, 32 tokens, heights 1 / 2 / 3 / 4 / 6: 28.5 /
// 21.7 / 25.1 / 16.6 / 21.9 us, 4 chosen.
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
// (us, this kernel against that one):
//  * up to 32 tokens always: 7B layer, f16, o 8.8 / 14.8 (17 tokens), 11.5 / 15.7
//    (32), q+k+v 16.6 / 25.2, gate+up 23.1 / 37.6, 70B gate+up 108 / 112, down 64
//    / 75 (32);
//  * to 64 tokens from the tiled layout, unless the batch has the 32768 rows from
//    which the tiled product no longer splits K: bf16, 64 tokens, o 17 / 24,
//    gate+up 38 / 47, 70B down 98 / 110, but 70B gate+up (57344 rows) 141 / 122;
//  * to 64 tokens from row-major activations while a CU's share of them, rounds *
//    M * K, is below 2^18 (48 tokens: gate+up 28.3 / 39.2; K = 11008 36 / 26; 64
//    tokens: K = 2048, 11264 rows 15.4 / 21.3, o 19.7 / 18.2).
// Every workgroup reads all activations, row-major ones in pieces of 64 bytes at
// 15 bytes a clock and CU, the tiled layout at more than twice that, so above a
// share of 3 * 2^16 (2^18 up to 32 tokens) a copy into it (a launch of about 2
// us) pays: f16, copied against row-major, 64 tokens: o 12.7 / 19.7, q+k+v 21.4 /
// 25.3, gate+up 33.6 / 44.8 (and 18.2, 27.2, 40.9 on the tiled product); 24
// tokens: K = 11008 17.4 / 21.3, but K = 8192 (a share of 3 * 2^16) 23.7 / 21.1.
MidPlan mid_plan(const int64_t* N, int count, int64_t K, int64_t M, bool bf16, bool room) {
    if (M <= kSkinnyMaxM || M > kMidMaxM) return {false, false};
    if ((M + 15) / 16 * 16 * K * 2 > kMaxBufferBytes) return {false, false};  // (32-bit offsets: the tiled product slices)
    int64_t rows = 0, rounds = 1;
    for (int i = 0; i < count; ++i) rows += N[i];
    mid_height(N, count, K, M, rounds);
    const int64_t share = rounds * M * K;
    const bool copy = bf16 || (room && share >= (M <= 32 ? 1 << 18 : 3 << 16));
    return {M <= 32 || (copy ? rows < 32768 : share < (1 << 18)), copy};
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
