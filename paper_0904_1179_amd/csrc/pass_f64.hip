// pass_f64.hip -- the heat-bath passes of FP64 links.
#include "pass_kernels.h"

namespace su3hb {

hipError_t launch_pass_f64(const PassArgs &a) { return launch_pass_r<double>(a); }
hipError_t launch_batch_f64(const BatchArgs &b) { return launch_batch_r<double>(b); }

}  // namespace su3hb
