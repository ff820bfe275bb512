// Instances of conv_small_kernel for one storage type.
#include "conv_small.h"
namespace octo {
hipError_t launch_small_f32(int which, const ConvArgs& a, int num_cu, hipStream_t s, int* kernel_id, const ConvTiming& tm) { return launch_small<float>(which, a, num_cu, s, kernel_id, tm); }
}  // namespace octo
