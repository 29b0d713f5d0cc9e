// Block kernel: the variants of 6-bit weights.
#include "abq_block_kernels.h"

namespace abq {
ABQ_BLOCK_LAUNCH(6) { return block_launch<6>(prm, shape, s); }
}  // namespace abq
