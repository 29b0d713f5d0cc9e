// Block kernel: the variants of 3-bit weights.
#include "abq_block_kernels.h"

namespace abq {
ABQ_BLOCK_LAUNCH(3) { return block_launch<3>(prm, shape, s); }
}  // namespace abq
