// Instances of conv_flow_kernel for one storage type.
#include "conv_flow.h"
#include "conv_flow_choice.h"
namespace octo {
hipError_t launch_flow_f8(int which, const ConvArgs& a, int num_cu, hipStream_t s, int* kernel_id, const ConvTiming& tm) { return launch_flow<f8>(which, a, num_cu, s, kernel_id, tm); }
}  // namespace octo
