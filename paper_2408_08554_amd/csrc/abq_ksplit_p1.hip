// Kernel instantiations of the K-split prefill kernel for weights of 1 bits.
#include "abq_ksplit_kernels.h"

namespace abq {

hipError_t ksplit_launch_p1(const KsplitParams& prm, int shape, bool raw, bool gq, hipStream_t s) { return ks_launch_p<1>(prm, shape, raw, gq, s); }

}  // namespace abq
