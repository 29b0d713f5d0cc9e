// Block kernels: the variants of 4-bit weights.
#include "abq_block_g128_kernels.h"

namespace abq {
ABQ_BLOCK_LAUNCH(4) { return block_launch<4>(prm, shape, s); }
ABQ_BLOCK_G128_LAUNCH(4) { return block_g128_launch<4>(prm, shape, s); }
}  // namespace abq
