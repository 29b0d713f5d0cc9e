// Block kernel: the variants of 4-bit weights.
#include "abq_block_kernels.h"

namespace abq {
ABQ_BLOCK_LAUNCH(4) { return block_launch<4>(prm, shape, s); }
}  // namespace abq
