// Launch helpers of the fused covariance -> blocked matrix-core solve
// (fused_impl.h, bsolve_impl.h): dispatch over the covariance block columns,
// the steering class and the wave count.  Included by one translation unit
// per (precision, single or batched) so the instantiations build in
// parallel.
#pragma once

#include <type_traits>

#include "fused_impl.h"

namespace stap {
namespace bfused {


// register blocks per wave for NB block columns and NS steering blocks
constexpr int nsl(int NB, int NW) { return (NB * (NB + 1) / 2 + NW - 1) / NW; }
constexpr int nsm(int NB, int NS, int NW) { return (NS * NB + NW - 1) / NW; }
// Whether the corrected form exists: not for 6 block columns on four waves,
// which run where a tuned entry asked for them and never by default.
constexpr bool has_corrected(int NB, int NW) { return NB != 6 || NW == 8; }

template <int NB, int NS, int NW, int MODE>
hipError_t go1(const Dims& d, const float2* snap, const float2* steer, float2* w, int* info, hipStream_t st) {
  constexpr int L = nsl(NB, NW), M = nsm(NB, NS, NW);
  const dim3 grid(d.P * d.B), block(64 * NW);
  if (d.refine == 0)
    hipLaunchKernelGGL((bfused_kernel<NB, NS, L, M, NW, MODE, kPlain>), grid, block, 0, st, snap, steer, w, info, d);
  else if (d.corr && has_corrected(NB, NW))
    hipLaunchKernelGGL((bfused_kernel<NB, NS, L, M, NW, MODE, has_corrected(NB, NW) ? kCorrected : kRefined>), grid, block,
                       0, st, snap, steer, w, info, d);
  else
    hipLaunchKernelGGL((bfused_kernel<NB, NS, L, M, NW, MODE, kRefined>), grid, block, 0, st, snap, steer, w, info, d);
  return hipGetLastError();
}

template <int NB, int NS, int NW, int MODE>
hipError_t gob(const ProbDesc* desc, int n, long long total, int level, hipStream_t st, unsigned long long* queue) {
  constexpr int L = nsl(NB, NW), M = nsm(NB, NS, NW);
  // enough workgroups to fill every CU a few times over, never more than systems
  const long long want = 256LL * (16 / NW);
  const dim3 grid((unsigned)(total < want ? total : want)), block(64 * NW);
  if (level == kPlain)
    hipLaunchKernelGGL((bfused_batched_kernel<NB, NS, L, M, NW, MODE, kPlain>), grid, block, 0, st, desc, n, total,
                       queue);
  else if (level == kCorrected && has_corrected(NB, NW))
    hipLaunchKernelGGL((bfused_batched_kernel<NB, NS, L, M, NW, MODE, has_corrected(NB, NW) ? kCorrected : kRefined>),
                       grid, block, 0, st, desc, n, total, queue);
  else
    hipLaunchKernelGGL((bfused_batched_kernel<NB, NS, L, M, NW, MODE, kRefined>), grid, block, 0, st, desc, n, total,
                       queue);
  return hipGetLastError();
}

// Waves per system: one or two where the system has one or two block columns
// (their few blocks leave more waves idle at every barrier), four up to 64
// DOF, and at 96 DOF four or eight as the variant asks.  Every count gives
// the same bits.
constexpr int nw_of(int NB) { return NB == 1 ? 1 : NB == 2 ? 2 : 4; }

// one switch for the single-cube and batched launches
template <int MODE, class F>
hipError_t pick(int D, int S, int waves, F&& f) {
  const int nb = (D + 15) / 16;
  const int ns = S <= 16 ? 1 : S <= 32 ? 2 : 4;
  auto by_s = [&](auto nbc, auto nwc) -> hipError_t {
    constexpr int NB = decltype(nbc)::value, NW = decltype(nwc)::value;
    if (ns == 1) return f(std::integral_constant<int, NB>{}, std::integral_constant<int, 1>{}, nwc);
    if (ns == 2) return f(std::integral_constant<int, NB>{}, std::integral_constant<int, 2>{}, nwc);
    return f(std::integral_constant<int, NB>{}, std::integral_constant<int, 4>{}, nwc);
  };
  using W4 = std::integral_constant<int, 4>;
  using W8 = std::integral_constant<int, 8>;
  switch (nb) {
    case 1: return by_s(std::integral_constant<int, 1>{}, std::integral_constant<int, nw_of(1)>{});
    case 2: return by_s(std::integral_constant<int, 2>{}, std::integral_constant<int, nw_of(2)>{});
    case 3: return by_s(std::integral_constant<int, 3>{}, W4{});
    case 4: return by_s(std::integral_constant<int, 4>{}, W4{});
    case 5: case 6:
      return waves == 8 ? by_s(std::integral_constant<int, 6>{}, W8{}) : by_s(std::integral_constant<int, 6>{}, W4{});
    case 7: case 8: return by_s(std::integral_constant<int, 8>{}, W8{});
  }
  return hipErrorInvalidValue;
}

// Whether pick() takes eight waves for D and the requested waves.
inline bool pick_eight(int D, int waves) {
  const int nb = (D + 15) / 16;
  return nb > 6 || (nb > 4 && waves == 8);
}

// One-cube launches of the shapes that run on eight waves, or of the others
// (in separate translation units, which build in parallel).
template <int MODE, bool EIGHT>
hipError_t single(const Dims& d, const float2* snap, const float2* steer, float2* w, int* info, hipStream_t st,
                  int waves) {
  return pick<MODE>(d.D, d.S, waves, [&](auto nb, auto ns, auto nw) -> hipError_t {
    if constexpr ((decltype(nw)::value == 8) == EIGHT)
      return go1<decltype(nb)::value, decltype(ns)::value, decltype(nw)::value, MODE>(d, snap, steer, w, info, st);
    else
      return hipErrorInvalidValue;
  });
}

template <int MODE>
hipError_t batched(const ProbDesc* desc, int n, long long total, int max_dof, int max_steer, int level, int waves,
                   hipStream_t st, unsigned long long* queue) {
  return pick<MODE>(max_dof, max_steer, waves, [&](auto nb, auto ns, auto nw) {
    return gob<decltype(nb)::value, decltype(ns)::value, decltype(nw)::value, MODE>(desc, n, total, level, st,
                                                                                   queue);
  });
}

}  // namespace bfused
}  // namespace stap
