// Block kernel: the variants of 2-bit weights.
#include "abq_block_kernels.h"

namespace abq {
ABQ_BLOCK_LAUNCH(2) { return block_launch<2>(prm, shape, s); }
}  // namespace abq
