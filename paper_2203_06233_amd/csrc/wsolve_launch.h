// Kernel and launch of the one-wave stage solve for one steering class;
// included by wsolve_s{1,2}.hip.
#pragma once

#include "kernels.h"
#include "wsolve_impl.h"

namespace stap {
namespace wsv {

// Waves per SIMD that the blocks of a system leave registers for: eight a
// block and about 60 to work with.  With 6 block columns 94 registers spill.
constexpr int wsolve_waves(int NB, int NS) {
  const int blocks = NB * (NB + 1) / 2 + steer_group(NB, NS) * NB;
  return blocks <= 8 ? 4 : blocks <= 13 ? 3 : 2;
}

template <int NB, int NS>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(wsolve_waves(NB, NS))))
void wsolve_kernel(const float2* __restrict__ cov, const float2* __restrict__ steer,
                                                    float2* __restrict__ wout, int* __restrict__ info_out, Dims d) {
  __shared__ __align__(16) float2 lds[WsLds<NB>::COMPLEX];
  const int sys = blockIdx.x;
  wsolve_system<NB, NS>(cov + (long long)sys * d.D * d.D, steer + steer_offset(d, sys), wout + (long long)sys * d.S * d.D,
                                info_out ? info_out + sys : nullptr, d, lds);
}

template <int NB, int NS>
hipError_t go(const Dims& d, const float2* cov, const float2* steer, float2* w, int* info, hipStream_t st) {
  hipLaunchKernelGGL((wsolve_kernel<NB, NS>), dim3(d.P * d.B), dim3(64), 0, st, cov, steer, w, info, d);
  return hipGetLastError();
}

template <int NS>
hipError_t by_nb(const Dims& d, const float2* cov, const float2* steer, float2* w, int* info, hipStream_t st) {
  switch ((d.D + 15) / 16) {
    case 1: return go<1, NS>(d, cov, steer, w, info, st);
    case 2: return go<2, NS>(d, cov, steer, w, info, st);
    case 3: return go<3, NS>(d, cov, steer, w, info, st);
    case 4: return go<4, NS>(d, cov, steer, w, info, st);
    case 5: return go<5, NS>(d, cov, steer, w, info, st);
    case 6: return go<6, NS>(d, cov, steer, w, info, st);
  }
  return hipErrorInvalidValue;
}

}  // namespace wsv
}  // namespace stap
