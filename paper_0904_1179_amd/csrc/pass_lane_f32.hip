// pass_lane_f32.hip -- the one-wave heat-bath passes of FP32 links.
#include "pass_lane.h"

namespace su3hb {

hipError_t launch_lane_f32(const PassArgs &a) { return launch_lane_r<float>(a); }
hipError_t launch_lane_batch_f32(const BatchArgs &b) { return launch_lane_batch_r<float>(b); }

}  // namespace su3hb
