// Block kernel: the variants of 7-bit weights.
#include "abq_block_kernels.h"

namespace abq {
ABQ_BLOCK_LAUNCH(7) { return block_launch<7>(prm, shape, s); }
}  // namespace abq
