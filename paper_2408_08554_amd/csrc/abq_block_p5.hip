// Block kernels: the variants of 5-bit weights.
#include "abq_block_g128_kernels.h"

namespace abq {
ABQ_BLOCK_LAUNCH(5) { return block_launch<5>(prm, shape, s); }
ABQ_BLOCK_G128_LAUNCH(5) { return block_g128_launch<5>(prm, shape, s); }
}  // namespace abq
