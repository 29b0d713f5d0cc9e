// Block kernel: the variants of 5-bit weights.
#include "abq_block_kernels.h"

namespace abq {
ABQ_BLOCK_LAUNCH(5) { return block_launch<5>(prm, shape, s); }
}  // namespace abq
