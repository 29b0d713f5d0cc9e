// Block kernel: the variants of 1-bit weights.
#include "abq_block_kernels.h"

namespace abq {
ABQ_BLOCK_LAUNCH(1) { return block_launch<1>(prm, shape, s); }
}  // namespace abq
