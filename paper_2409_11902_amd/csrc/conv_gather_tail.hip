// The gather GEMM with a weight gradient's slice sum in workgroups of its launch.
#include "conv_gather.h"

namespace cac {

hipError_t launch_conv_gather_tail(const GatherParams &p, int variant, hipStream_t st) { return launch_gather_variant<true>(p, variant, st); }

} // namespace cac
