// Batch products for 17 to 64 tokens: the codes-only kernels (row-shared pairs).
#include "midbatch_kernel.hpp"

namespace unisvq {

hipError_t mid_launch_shared(const MidBatch& b, int rb, int blocks, hipStream_t s) {
    return mid_launch_format<true>(b, rb, blocks, s);
}

}  // namespace unisvq
