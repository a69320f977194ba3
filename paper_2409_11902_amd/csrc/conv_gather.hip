// The gather GEMM by itself.
#include "conv_gather.h"

namespace cac {

hipError_t launch_conv_gather(const GatherParams &p, int variant, hipStream_t st) { return launch_gather_variant<false>(p, variant, st); }

} // namespace cac
