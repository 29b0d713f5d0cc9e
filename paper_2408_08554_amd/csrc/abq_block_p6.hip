// Block kernels: the variants of 6-bit weights.
#include "abq_block_g128_kernels.h"

namespace abq {
ABQ_BLOCK_LAUNCH(6) { return block_launch<6>(prm, shape, s); }
ABQ_BLOCK_G128_LAUNCH(6) { return block_g128_launch<6>(prm, shape, s); }
}  // namespace abq
