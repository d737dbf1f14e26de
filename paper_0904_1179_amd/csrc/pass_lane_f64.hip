// pass_lane_f64.hip -- the one-wave heat-bath passes of FP64 links.
#include "pass_lane.h"

namespace su3hb {

hipError_t launch_lane_f64(const PassArgs &a) { return launch_lane_r<double>(a); }
hipError_t launch_lane_batch_f64(const BatchArgs &b) { return launch_lane_batch_r<double>(b); }

}  // namespace su3hb
