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
//
// The split covers the values that three BF16 terms hold: an infinite value,
// or one that rounds to infinity in BF16 (above 3.39e38), leaves NaN in its
// second term, and the lower terms of a value below 2^-110 are denormal, which
// the matrix cores flush (relative error 2.7e-5 at 1e-36).  Tiles where that
// can show are formed again from the FP32 operands on v_mfma_f32_16x16x4_f32
// once the wave has done its tiles: those with an output that is not finite,
// or below 2^-46 and not zero, and all of a system with weights of 2^40 and
// more or a pair of them that are below 2^-95 and not zero.  Below 2^40 a cell
// whose values are all under 2^-95 gives outputs under 2^-46 (192 DOF), so no
// look at the samples is needed (one costs 4 %); forming the tiles again in the
// loop itself takes the registers of the others (48 DOF, 32 vectors, 4096
// blocks of 48 cells: 31 -> 40 us).
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


// Whether a pair of weights is outside what the split and the test on its
// outputs cover: 2^40 or more, or not zero and nothing of 2^-95 or more.
__device__ __forceinline__ bool odd_pair(float2 a, float2 b) {
  const float top = fmaxf(fmaxf(fabsf(a.x), fabsf(a.y)), fmaxf(fabsf(b.x), fabsf(b.y)));
  return (top >= 0x1p40f) | ((top < 0x1p-95f) & (top != 0.f));
}

// The lane's outputs of a range tile, rows s of steering tile t in register i:
// power (and y) at o + s R.  Returns whether one is not finite, or below 2^-46
// and not zero.
template <int ST>
__device__ __forceinline__ bool store_tile(const floatx4 (&re)[ST], const floatx4 (&im)[ST], float* __restrict__ power,
                                           float2* __restrict__ yout, long long o, int S, int R, int lane) {
  constexpr unsigned int kLow = (127 - 46) << 23, kInf = 0x7f800000u;
  unsigned int out = 0;
#pragma unroll
  for (int t = 0; t < ST; ++t)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int s = t * 16 + 4 * (lane >> 4) + i;
      if (s < S) {
        const long long at = o + (long long)s * R;
        power[at] = re[t][i] * re[t][i] + im[t][i] * im[t][i];
        if (yout) yout[at] = make_float2(re[t][i], im[t][i]);
        const unsigned int u = __float_as_uint(fabsf(re[t][i]) + fabsf(im[t][i]));
        out = max(out, u == 0 ? 0u : u - kLow);
      }
    }
  return out >= kInf - kLow;
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
  __shared__ int odd_w[NW];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int k = sys / d.B, b = sys - (sys / d.B) * d.B;
  const int D = d.D, S = d.S, N = d.N;
  const float2* W = wts + (long long)sys * S * D;
  bool odd = false;
  for (int e = tid; e < SP * (DP / 2); e += 64 * NW) {
    const int s = e / (DP / 2), q = 2 * (e % (DP / 2));
    float2 w0 = make_float2(0.f, 0.f), w1 = w0;
    if (s < S) {
      if (q < D) w0 = W[s * D + q];
      if (q + 1 < D) w1 = W[s * D + q + 1];
    }
    odd |= odd_pair(w0, w1);
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
  odd = __any(odd);
  if (lane == 0) odd_w[wave] = odd;
  __syncthreads();
  const uint4* wp4 = reinterpret_cast<const uint4*>(wp);
  const float2* X = snap + (long long)k * D * d.R + (long long)b * N;
  const int ntile = (N + 15) / 16;
  constexpr int PA[5] = {0, 1, 0, 2, 1};
  constexpr int PB[5] = {1, 0, 2, 0, 1};
  // Each wave takes one range tile at a time: two tiles would share the
  // weights' fragments, but cost the registers of a workgroup per compute
  // unit (1.68 against 1.00 ms on the 32 x 256 x 16384 cube).
  unsigned long long again = 0;  // bit rt / NW (mod 64): tile rt is to be formed from FP32
#pragma unroll
  for (int w = 0; w < NW; ++w) again = odd_w[w] ? ~0ULL : again;
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
#pragma unroll
    for (int t = 0; t < ST; ++t) {
      accR[t] += corR[t];
      accI[t] += corI[t];
    }
    bool out = false;
    if (live) out = store_tile<ST>(accR, accI, power, yout, (long long)k * S * d.R + (long long)b * N + r, S, d.R, lane);
    if (__any(out)) again |= 1ULL << (rt / NW & 63);
  }
  if (!again) return;
  const int l = lane_tid() & 63;  // apart from the first loop's: nothing is kept live for this
  for (int rt = wave; rt < ntile; rt += NW) {
    if (!(again >> (rt / NW & 63) & 1)) continue;
    const int r = rt * 16 + (l & 15);
    const bool live = r < N;
    floatx4 re[ST], im[ST];
#pragma unroll
    for (int t = 0; t < ST; ++t) re[t] = im[t] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
    for (int q0 = 0; q0 < D; q0 += 4) {
      const int q = q0 + (l >> 4);
      const float2 x = live && q < D ? X[(long long)q * d.R + r] : make_float2(0.f, 0.f);
#pragma unroll
      for (int t = 0; t < ST; ++t) {
        const int s = t * 16 + (l & 15);
        const float2 w = s < S && q < D ? W[s * D + q] : make_float2(0.f, 0.f);
        re[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(w.x, x.x, re[t], 0, 0, 0);
        re[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(w.y, x.y, re[t], 0, 0, 0);
        im[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(w.x, x.y, im[t], 0, 0, 0);
        im[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(-w.y, x.x, im[t], 0, 0, 0);
      }
    }
    if (live) store_tile<ST>(re, im, power, yout, (long long)k * S * d.R + (long long)b * N + r, S, d.R, l);
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
