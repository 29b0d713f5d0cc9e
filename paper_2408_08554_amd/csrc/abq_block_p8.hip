// Block kernel: the variants of 8-bit weights.
#include "abq_block_kernels.h"

namespace abq {
ABQ_BLOCK_LAUNCH(8) { return block_launch<8>(prm, shape, s); }
}  // namespace abq
