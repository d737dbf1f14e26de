// pass_f32.hip -- the heat-bath passes of FP32 links.
#include "pass_kernels.h"

namespace su3hb {

hipError_t launch_pass_f32(const PassArgs &a) { return launch_pass_r<float>(a); }
hipError_t launch_batch_f32(const BatchArgs &b) { return launch_batch_r<float>(b); }

}  // namespace su3hb
