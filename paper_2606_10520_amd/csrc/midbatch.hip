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
// (us, this kernel against that one; each with its bf16 pre-pass where there
// is one):
//  * up to 32 tokens always: 7B layer o 8.8 / 14.8 (17 tokens), 11.5 / 15.7
//    (32), q+k+v 16.6 / 25.2, gate+up 23.1 / 37.6, down 25.5 / 25.6 (32), 70B
//    gate+up 108 / 112, down 64 / 75 (32);
//  * tiled activations to 64 tokens, unless the batch has the 32768 rows from
//    which the tiled product no longer splits K: 64 tokens o 17 / 24, gate+up 38
//    / 47, 70B down 98 / 110, but 70B gate+up (57344 rows) 141 / 122;
//  * row-major activations above 32 tokens, read in pieces of 64 bytes by every
//    workgroup, while a CU's share is small: rounds * M * K below 2^18 (48
//    tokens, K = 4096: o 15.5 / 17.1, gate+up 28.3 / 39.2; at 64 tokens o 19.7 /
//    18.2, gate+up 44.8 / 40.9; 48 tokens, K = 11008 36 / 26; 64 tokens, K = 2048,
//    11264 rows 15.4 / 21.3).
bool mid_serves(const int64_t* N, int count, int64_t K, int64_t M, bool tiled) {
    if (M <= kSkinnyMaxM || M > kMidMaxM) return false;
    if ((M + 15) / 16 * 16 * K * 2 > kMaxBufferBytes) return false;  // (32-bit offsets: the tiled product slices)
    if (M <= 32) return true;
    int64_t rows = 0, rounds = 1;
    for (int i = 0; i < count; ++i) rows += N[i];
    if (tiled) return rows < 32768;
    mid_height(N, count, K, M, rounds);
    return rounds * M * K < (1 << 18);
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
