// Fused covariance -> blocked matrix-core solve, FP32 covariance products:
// the one-cube launches, 8-wave shapes here, the others in
// bfused_f32_w4.hip.
#include "bfused_launch.h"

namespace stap {

hipError_t launch_bfused_f32_w4(const Dims& d, const float2* snap, const float2* steer, float2* w, int* info,
                                 hipStream_t st, int waves);

hipError_t launch_bfused_f32(const Dims& d, const float2* snap, const float2* steer, float2* w, int* info,
                              hipStream_t st, int waves) {
  if (!bfused::pick_eight(d.D, waves)) return launch_bfused_f32_w4(d, snap, steer, w, info, st, waves);
  return bfused::single<0, true>(d, snap, steer, w, info, st, waves);
}

}  // namespace stap
