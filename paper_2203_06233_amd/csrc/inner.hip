// Weight x snapshot inner products and output power (statement U applied to
// the adaptive weights):
//
//   y[k][s][r] = w_{k,b(r),s}^H X[k][:, r],   power = |y|^2.
//
// One workgroup per system (k, b): a complex (S x D) x (D x N) product,
//   Re y = Wr.Xr + Wi.Xi,   Im y = Wr.Xi - Wi.Xr.
// The weights of the system are staged once in LDS; each wave owns a set of
// 16-cell range tiles and all steering tiles, so every snapshot element is
// read from HBM exactly once, coalesced along range.
//
// On every precision path weights and snapshots are split exactly into three
// BF16 terms each; the six products hh, hm, mh, hl, lh, mm run on
// v_mfma_f32_16x16x32_bf16, the hh term in its own accumulator, so the output
// keeps FP32-level error (the filter output cancels the clutter, so a single
// BF16 term would not).  FP32 MFMA, the form the plain path had before,
// occupies the vector ALU 2.7 times as long for the same products; the split
// leaves the pass to HBM.  It is also the more exact form: relative error of the
// power against 64 bits 2.9e-7 -> 0.95e-7 at 12 DOF, 9.8e-7 -> 3.2e-7 at 96,
// 1.6e-6 -> 3.7e-7 at 192 (FP32 MFMA -> split).
#include <type_traits>

#include "common.h"
#include "kernels.h"

namespace stap {

namespace {

__device__ __forceinline__ floatx4 mfma_bf16x(uint4 a, uint4 b, floatx4 c) {
  typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf, a), __builtin_bit_cast(v8bf, b),
                                                 c, 0, 0, 0);
}


// One system on NW waves.  LDS holds the weights as six planes
// [re h, re m, re l, im h, im m, im l][s][d] (d padded to DP, pitch DP + 8).
template <int ST, int DP, int NW>
__device__ __forceinline__ void inner_system(const float2* __restrict__ wts, const float2* __restrict__ snap,
                                             float* __restrict__ power, float2* __restrict__ yout, const Dims& d,
                                             int sys) {
  constexpr int SP = ST * 16;
  constexpr int PITCH = DP + 8;              // bf16 units per row
  constexpr int PS = SP * PITCH / 2;         // plane stride in uint32
  __shared__ __align__(16) unsigned int wp[6 * PS];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int k = sys / d.B, b = sys - (sys / d.B) * d.B;
  const int D = d.D, S = d.S, N = d.N;
  const float2* W = wts + (long long)sys * S * D;
  for (int e = tid; e < SP * (DP / 2); e += 64 * NW) {
    const int s = e / (DP / 2), q = 2 * (e % (DP / 2));
    float2 w0 = make_float2(0.f, 0.f), w1 = w0;
    if (s < S) {
      if (q < D) w0 = W[s * D + q];
      if (q + 1 < D) w1 = W[s * D + q + 1];
    }
    unsigned int h, m, l;
    const int o = s * (PITCH / 2) + q / 2;
    split3x2(w0.x, w1.x, h, m, l);
    wp[0 * PS + o] = h;
    wp[1 * PS + o] = m;
    wp[2 * PS + o] = l;
    split3x2(w0.y, w1.y, h, m, l);
    wp[3 * PS + o] = h;
    wp[4 * PS + o] = m;
    wp[5 * PS + o] = l;
  }
  __syncthreads();
  const uint4* wp4 = reinterpret_cast<const uint4*>(wp);
  const float2* X = snap + (long long)k * D * d.R + (long long)b * N;
  const int ntile = (N + 15) / 16;
  constexpr int PA[5] = {0, 1, 0, 2, 1};
  constexpr int PB[5] = {1, 0, 2, 0, 1};
  // Each wave takes one range tile at a time: two tiles would share the
  // weights' fragments, but cost the registers of a workgroup per compute
  // unit (1.68 against 1.00 ms on the 32 x 256 x 16384 cube).
  for (int rt = wave; rt < ntile; rt += NW) {
    const int r = rt * 16 + (lane & 15);
    const bool live = r < N;
    floatx4 accR[ST], accI[ST], corR[ST], corI[ST];
#pragma unroll
    for (int t = 0; t < ST; ++t) {
      accR[t] = floatx4{0.f, 0.f, 0.f, 0.f};
      accI[t] = accR[t];
      corR[t] = accR[t];
      corI[t] = accR[t];
    }
#pragma unroll 1
    for (int q0 = 0; q0 < DP; q0 += 32) {
      // B operand: X[q0 + 8*(lane/16) + j][r], j = 0..7, split into 3 terms
      unsigned int xb[6][4];
#pragma unroll
      for (int j = 0; j < 8; j += 2) {
        const int q = q0 + 8 * (lane >> 4) + j;
        const float2 x0 = (live && q < D) ? X[(long long)q * d.R + r] : make_float2(0.f, 0.f);
        const float2 x1 = (live && q + 1 < D) ? X[(long long)(q + 1) * d.R + r] : make_float2(0.f, 0.f);
        split3x2(x0.x, x1.x, xb[0][j / 2], xb[1][j / 2], xb[2][j / 2]);
        split3x2(x0.y, x1.y, xb[3][j / 2], xb[4][j / 2], xb[5][j / 2]);
      }
      uint4 Bv[6];
#pragma unroll
      for (int p = 0; p < 6; ++p) Bv[p] = make_uint4(xb[p][0], xb[p][1], xb[p][2], xb[p][3]);
#pragma unroll
      for (int t = 0; t < ST; ++t) {
        const int o = (t * 16 + (lane & 15)) * (PITCH / 8) + q0 / 8 + (lane >> 4);
        uint4 A[6];
#pragma unroll
        for (int p = 0; p < 6; ++p) A[p] = wp4[p * (PS / 4) + o];
        // Re += Wr Xr + Wi Xi ;  Im += Wr Xi - Wi Xr
        accR[t] = mfma_bf16x(A[0], Bv[0], accR[t]);
        accR[t] = mfma_bf16x(A[3], Bv[3], accR[t]);
        accI[t] = mfma_bf16x(A[0], Bv[3], accI[t]);
        accI[t] = mfma_bf16x(negbf8(A[3]), Bv[0], accI[t]);
#pragma unroll
        for (int u = 0; u < 5; ++u) {
          corR[t] = mfma_bf16x(A[PA[u]], Bv[PB[u]], corR[t]);
          corR[t] = mfma_bf16x(A[3 + PA[u]], Bv[3 + PB[u]], corR[t]);
          corI[t] = mfma_bf16x(A[PA[u]], Bv[3 + PB[u]], corI[t]);
          corI[t] = mfma_bf16x(negbf8(A[3 + PA[u]]), Bv[PB[u]], corI[t]);
        }
      }
    }
    if (!live) continue;
    const long long rr = (long long)b * N + r;
#pragma unroll
    for (int t = 0; t < ST; ++t)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int s = t * 16 + 4 * (lane >> 4) + i;
        if (s < S) {
          const float re = accR[t][i] + corR[t][i], im = accI[t][i] + corI[t][i];
          const long long o = ((long long)k * S + s) * d.R + rr;
          power[o] = re * re + im * im;
          if (yout) yout[o] = make_float2(re, im);
        }
      }
  }
}

// Waves per system.  Blocks of up to 16 or 32 cells have one or two range
// tiles and take one or two waves (four leave the others idle behind the
// staging: 49 -> 41 us on 43648 systems of 24 cells, 12 DOF); above 128 DOF
// the weights fill the LDS of a compute unit from three steering tiles on, and
// eight waves keep loads in flight (192 DOF, 64 steering vectors: 0.68 ms with
// FP32 MFMA on four waves, 0.35 so).
constexpr int waves_of(int ST, int DP, int N) {
  return N <= 16 ? 1 : N <= 32 ? 2 : DP > 128 && ST > 2 && N > 64 ? 8 : 4;
}
// Register budgets that fit without spills: 128 with one steering tile, 168
// with two from 64 DOF on (164 at 96 DOF): four and three 256-thread
// workgroups per compute unit, for the loads in flight that this
// bandwidth-bound pass needs.
constexpr int min_waves(int ST, int DP, int NW) {
  return ST == 1 ? 4 : ST == 2 && DP >= 64 && NW <= 4 ? 3 : 1;
}

template <int ST, int DP, int NW>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(min_waves(ST, DP, NW))))
void inner_kernel(const float2* __restrict__ wts, const float2* __restrict__ snap, float* __restrict__ power,
                  float2* __restrict__ yout, Dims d) {
  inner_system<ST, DP, NW>(wts, snap, power, yout, d, blockIdx.x);
}

// Batched: one workgroup per system of every cube of the table.
template <int ST, int DP, int NW>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(min_waves(ST, DP, NW))))
void inner_batched_kernel(const ProbDesc* __restrict__ desc, int n) {
  const long long g = blockIdx.x;
  int lo = 0, hi = n - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (desc[mid].sys_begin <= g) lo = mid;
    else hi = mid - 1;
  }
  const ProbDesc& pd = desc[lo];
  const Dims d = pd.d;
  inner_system<ST, DP, NW>(pd.w, pd.snap, pd.power, nullptr, d, (int)(g - pd.sys_begin));
}

template <class F>
hipError_t by_dof(int D, F&& f) {
  if (D <= 32) return f(std::integral_constant<int, 32>{});
  if (D <= 64) return f(std::integral_constant<int, 64>{});
  if (D <= 96) return f(std::integral_constant<int, 96>{});
  if (D <= 128) return f(std::integral_constant<int, 128>{});
  return f(std::integral_constant<int, 192>{});
}
template <class F>
hipError_t by_steer(int S, F&& f) {
  switch ((S + 15) / 16) {
    case 1: return f(std::integral_constant<int, 1>{});
    case 2: return f(std::integral_constant<int, 2>{});
    case 3: return f(std::integral_constant<int, 3>{});
    case 4: return f(std::integral_constant<int, 4>{});
  }
  return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_inner_batched(const ProbDesc* desc, int n, long long total_sys, int max_dof, int max_steer,
                                hipStream_t st) {
  if (max_dof > 128 || total_sys <= 0) return hipErrorInvalidValue;
  return by_steer(max_steer, [&](auto sc) {
    return by_dof(max_dof, [&](auto dc) -> hipError_t {
      constexpr int ST = sc.value, DP = dc.value;
      if constexpr (DP <= 128)
        hipLaunchKernelGGL((inner_batched_kernel<ST, DP, 4>), dim3((unsigned)total_sys), dim3(256), 0, st, desc, n);
      return hipGetLastError();
    });
  });
}

hipError_t launch_inner(const Dims& d, const float2* w, const float2* snap, float* power, float2* y,
                        hipStream_t st) {
  return by_steer(d.S, [&](auto sc) {
    return by_dof(d.D, [&](auto dc) -> hipError_t {
      constexpr int ST = sc.value, DP = dc.value;
      const dim3 g(d.P * d.B);
      const int nw = waves_of(ST, DP, d.N);
      if (nw == 1) hipLaunchKernelGGL((inner_kernel<ST, DP, 1>), g, dim3(64), 0, st, w, snap, power, y, d);
      else if (nw == 2) hipLaunchKernelGGL((inner_kernel<ST, DP, 2>), g, dim3(128), 0, st, w, snap, power, y, d);
      else if (nw == 8) hipLaunchKernelGGL((inner_kernel<ST, DP, (DP > 128 ? 8 : 4)>), g, dim3(512), 0, st, w, snap, power, y, d);
      else hipLaunchKernelGGL((inner_kernel<ST, DP, 4>), g, dim3(256), 0, st, w, snap, power, y, d);
      return hipGetLastError();
    });
  });
}

}  // namespace stap
