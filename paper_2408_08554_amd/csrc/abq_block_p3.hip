// Block kernels: the variants of 3-bit weights.
#include "abq_block_g128_kernels.h"

namespace abq {
ABQ_BLOCK_LAUNCH(3) { return block_launch<3>(prm, shape, s); }
ABQ_BLOCK_G128_LAUNCH(3) { return block_g128_launch<3>(prm, shape, s); }
}  // namespace abq
