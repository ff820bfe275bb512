// Instances of conv_small_kernel for one storage type.
#include "conv_small.h"
namespace octo {
hipError_t launch_small_bf16(int which, const ConvArgs& a, int num_cu, hipStream_t s, int* kernel_id, const ConvTiming& tm) { return launch_small<__bf16>(which, a, num_cu, s, kernel_id, tm); }
hipError_t launch_small_group_bf16(const SmallGroup& g, hipStream_t s) { return launch_small_group_t<__bf16>(g, s); }
}  // namespace octo
