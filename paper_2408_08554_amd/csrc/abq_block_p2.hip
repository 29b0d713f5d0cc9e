// Block kernels: the variants of 2-bit weights.
#include "abq_block_g128_kernels.h"

namespace abq {
ABQ_BLOCK_LAUNCH(2) { return block_launch<2>(prm, shape, s); }
ABQ_BLOCK_G128_LAUNCH(2) { return block_g128_launch<2>(prm, shape, s); }
}  // namespace abq
