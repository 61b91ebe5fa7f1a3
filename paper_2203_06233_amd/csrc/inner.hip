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
// On every precision path (but for the small shapes of plain FP32 that
// f32_form() names) weights and snapshots are split exactly into three
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
// or with a cell whose outputs are all below 2^-46 and not all zero, and all of
// a system with weights of 2^40 and more or a pair of them that are below
// 2^-95 and not zero.  With weights below 2^40 a cell whose values are all
// under 2^-95 gives outputs under 2^-46 (192 DOF), so no look at the samples
// is needed (one costs 4 %).  Forming the tiles again in the loop itself takes
// the registers of the others (48 DOF, 32 vectors, 4096 blocks of 48 cells:
// 31 -> 40 us).  The mixed path up to 128 DOF, which never had any other form,
// goes without (GUARD): it would cost up to 7 % there.
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
// power (and y) at o + s R.  Returns whether one is not finite, or all are
// below 2^-46 and not all zero.
template <int ST>
__device__ __forceinline__ bool store_tile(const floatx4 (&re)[ST], const floatx4 (&im)[ST], float* __restrict__ power,
                                           float2* __restrict__ yout, long long o, int S, int R, int lane) {
  constexpr unsigned int kLow = (127 - 46) << 23, kInf = 0x7f800000u;
  unsigned int top = 0;
#pragma unroll
  for (int t = 0; t < ST; ++t)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int s = t * 16 + 4 * (lane >> 4) + i;
      if (s < S) {
        const long long at = o + (long long)s * R;
        power[at] = re[t][i] * re[t][i] + im[t][i] * im[t][i];
        if (yout) yout[at] = make_float2(re[t][i], im[t][i]);
        top = max(top, __float_as_uint(fabsf(re[t][i]) + fabsf(im[t][i])));
      }
    }
  return top >= kInf || (top < kLow && top != 0);
}

// One system on NW waves.  LDS holds the weights as six planes
// [re h, re m, re l, im h, im m, im l][s][d] (d padded to DP, pitch DP + 8).
template <int ST, int DP, int NW, bool GUARD>
__device__ __forceinline__ void inner_system(const float2* __restrict__ wts, const float2* __restrict__ snap,
                                             float* __restrict__ power, float2* __restrict__ yout, const Dims& d,
                                             int sys) {
  constexpr int SP = ST * 16;
  constexpr int PITCH = DP + 8;              // bf16 units per row
  constexpr int PS = SP * PITCH / 2;         // plane stride in uint32
  __shared__ __align__(16) unsigned int wp[6 * PS];
  __shared__ int odd_w[GUARD ? NW : 1];
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
    if (GUARD) odd |= odd_pair(w0, w1);
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
  if (GUARD) {
    odd = __any(odd);
    if (lane == 0) odd_w[wave] = odd;
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
  unsigned long long again = 0;  // bit rt / NW (mod 64): tile rt is to be formed from FP32
#pragma unroll
  for (int w = 0; w < (GUARD ? NW : 0); ++w) again = odd_w[w] ? ~0ULL : again;
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
    if (GUARD && __any(out)) again |= 1ULL << (rt / NW & 63);
  }
  if (!GUARD || !again) return;
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

// The same on v_mfma_f32_16x16x4_f32 with the FP32 weights in LDS ([s][d], odd
// pitch) and two range tiles per wave step; the snapshot loads of the next 16
// rows are issued before the products of the current ones.  Four waves.
template <int ST, int DP>
__device__ __forceinline__ void inner_f32_system(const float2* __restrict__ wts, const float2* __restrict__ snap,
                                                 float* __restrict__ power, float2* __restrict__ yout, const Dims& d,
                                                 int sys) {
  constexpr int SP = ST * 16, PITCH = DP + 1, RTW = 2;
  __shared__ float2 ws[SP * PITCH];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int k = sys / d.B, b = sys - (sys / d.B) * d.B;
  const int D = d.D, S = d.S, N = d.N;
  const float2* W = wts + (long long)sys * S * D;
  for (int e = tid; e < SP * DP; e += 256) {
    const int s = e / DP, q = e % DP;
    ws[s * PITCH + q] = (s < S && q < D) ? W[s * D + q] : make_float2(0.f, 0.f);
  }
  __syncthreads();
  const float2* X = snap + (long long)k * D * d.R + (long long)b * N;
  const int ntile = (N + 15) / 16;
  for (int rt0 = wave * RTW; rt0 < ntile; rt0 += 4 * RTW) {
    int r[RTW];
    bool live[RTW];
    floatx4 re[RTW][ST], im[RTW][ST];
#pragma unroll
    for (int w = 0; w < RTW; ++w) {
      r[w] = (rt0 + w) * 16 + (lane & 15);
      live[w] = r[w] < N;
#pragma unroll
      for (int t = 0; t < ST; ++t) re[w][t] = im[w][t] = floatx4{0.f, 0.f, 0.f, 0.f};
    }
    auto load = [&](int q0, float2 (&xv)[RTW][4]) {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int q = q0 + 4 * u + (lane >> 4);
#pragma unroll
        for (int w = 0; w < RTW; ++w)
          xv[w][u] = (live[w] && q < D) ? X[(long long)q * d.R + r[w]] : make_float2(0.f, 0.f);
      }
    };
    float2 cur[RTW][4], nxt[RTW][4];
    load(0, cur);
#pragma unroll 1
    for (int q0 = 0; q0 < DP; q0 += 16) {
      if (q0 + 16 < DP) load(q0 + 16, nxt);
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int q = q0 + 4 * u + (lane >> 4);
#pragma unroll
        for (int t = 0; t < ST; ++t) {
          const float2 wv = ws[(t * 16 + (lane & 15)) * PITCH + q];
#pragma unroll
          for (int w = 0; w < RTW; ++w) {
            re[w][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(wv.x, cur[w][u].x, re[w][t], 0, 0, 0);
            re[w][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(wv.y, cur[w][u].y, re[w][t], 0, 0, 0);
            im[w][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(wv.x, cur[w][u].y, im[w][t], 0, 0, 0);
            im[w][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(-wv.y, cur[w][u].x, im[w][t], 0, 0, 0);
          }
        }
      }
#pragma unroll
      for (int w = 0; w < RTW; ++w)
#pragma unroll
        for (int u = 0; u < 4; ++u) cur[w][u] = nxt[w][u];
    }
#pragma unroll
    for (int w = 0; w < RTW; ++w)
      if (live[w])
        store_tile<ST>(re[w], im[w], power, yout, (long long)k * S * d.R + (long long)b * N + r[w], S, d.R, lane);
  }
}

// Shapes of plain FP32 where the FP32 form is the faster one: the split works
// on 32 rows at a time, twice what up to 16 DOF fill, and its fragments leave
// two waves a SIMD from three steering tiles on (12 DOF, 48 vectors, 8192
// blocks of 96 cells: 97 us, split 183; 24 DOF, 48 vectors, 96 cells 1.26
// times as long split, 48 cells 0.88; 48 DOF, 64 vectors, 96 cells 1.37, 64
// cells 1.01).
constexpr bool f32_form(int D, int S, int N) {
  return S > 16 && ((D <= 16 && N > 16) || (D <= 32 && S > 32 && N > 64) || (D <= 48 && S > 48 && N > 64));
}

// Waves per system.  Blocks of up to 16 or 32 cells have one or two range
// tiles and leave most of four waves idle behind the staging of the weights
// (43648 systems of 24 cells, 12 DOF: 49 us on four, 41 on two).  But fewer
// waves also stage the weights more slowly, and where they fill the LDS, or the
// accumulators the registers, nothing else runs on the compute unit meanwhile:
// one wave up to 32 DOF (at 48 DOF, 32 vectors, 16 cells 74 us against 41 on
// four), two also with one steering tile (96 DOF, 24 cells: 0.72 of the time
// on four) and with four tiles up to 96 DOF (0.78; with two or three tiles
// 1.1 to 1.4); above 128 DOF the weights fill the LDS from three steering
// tiles on, and eight waves keep loads in flight (192 DOF, 64 steering
// vectors: 0.68 ms with FP32 MFMA on four waves, 0.35 so).
constexpr int waves_of(int ST, int DP, int N) {
  if (N <= 16 && DP <= 32) return 1;
  if (N <= 32 && (DP <= 32 || ST == 1 || (ST == 4 && DP <= 96))) return 2;
  return DP > 128 && ST > 2 && N > 64 ? 8 : 4;
}
// Register budgets that fit without spills: 128 with one steering tile, 168
// with two from 64 DOF on (164 at 96 DOF): four and three 256-thread
// workgroups per compute unit, for the loads in flight that this
// bandwidth-bound pass needs.
constexpr int min_waves(int ST, int DP, int NW) {
  return ST == 1 ? 4 : ST == 2 && DP >= 64 && NW <= 4 ? 3 : 1;
}

template <int ST, int DP, int NW, bool GUARD>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(min_waves(ST, DP, NW))))
void inner_kernel(const float2* __restrict__ wts, const float2* __restrict__ snap, float* __restrict__ power,
                  float2* __restrict__ yout, Dims d) {
  inner_system<ST, DP, NW, GUARD>(wts, snap, power, yout, d, blockIdx.x);
}

template <int ST, int DP>
__global__ __launch_bounds__(256) void inner_f32_kernel(const float2* __restrict__ wts, const float2* __restrict__ snap,
                                                        float* __restrict__ power, float2* __restrict__ yout, Dims d) {
  inner_f32_system<ST, DP>(wts, snap, power, yout, d, blockIdx.x);
}

// The cube of system g of the table.
__device__ __forceinline__ const ProbDesc& cube_of(const ProbDesc* __restrict__ desc, int n, long long g) {
  int lo = 0, hi = n - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (desc[mid].sys_begin <= g) lo = mid;
    else hi = mid - 1;
  }
  return desc[lo];
}

// Batched: one workgroup per system of every cube of the table.
template <int ST, int DP, int NW, bool GUARD>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(min_waves(ST, DP, NW))))
void inner_batched_kernel(const ProbDesc* __restrict__ desc, int n) {
  const ProbDesc& pd = cube_of(desc, n, blockIdx.x);
  const Dims d = pd.d;
  inner_system<ST, DP, NW, GUARD>(pd.w, pd.snap, pd.power, nullptr, d, (int)(blockIdx.x - pd.sys_begin));
}
template <int ST, int DP>
__global__ __launch_bounds__(256) void inner_f32_batched_kernel(const ProbDesc* __restrict__ desc, int n) {
  const ProbDesc& pd = cube_of(desc, n, blockIdx.x);
  const Dims d = pd.d;
  inner_f32_system<ST, DP>(pd.w, pd.snap, pd.power, nullptr, d, (int)(blockIdx.x - pd.sys_begin));
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

// f(steering tiles, padded DOF) of the shapes that f32_form() accepts.
template <class F>
hipError_t by_f32(int D, int S, F&& f) {
  return by_steer(S, [&](auto sc) -> hipError_t {
    constexpr int ST = sc.value;
    if constexpr (ST > 1) {
      if (D <= 16) return f(sc, std::integral_constant<int, 16>{});
      if constexpr (ST > 2)
        if (D <= 32) return f(sc, std::integral_constant<int, 32>{});
      if constexpr (ST > 3) return f(sc, std::integral_constant<int, 48>{});
    }
    return hipErrorInvalidValue;
  });
}

}  // namespace

// cells: block length of the cube with the most work.
hipError_t launch_inner_batched(const ProbDesc* desc, int n, long long total_sys, int max_dof, int max_steer, int prec,
                                int cells, hipStream_t st) {
  if (max_dof > 128 || total_sys <= 0) return hipErrorInvalidValue;
  if (prec == STAP_PREC_FP32 && f32_form(max_dof, max_steer, cells))
    return by_f32(max_dof, max_steer, [&](auto sc, auto dc) {
      hipLaunchKernelGGL((inner_f32_batched_kernel<sc.value, dc.value>), dim3((unsigned)total_sys), dim3(256), 0, st,
                         desc, n);
      return hipGetLastError();
    });
  return by_steer(max_steer, [&](auto sc) {
    return by_dof(max_dof, [&](auto dc) -> hipError_t {
      constexpr int ST = sc.value, DP = dc.value;
      if constexpr (DP <= 128) {
        const dim3 g((unsigned)total_sys), block(256);
        if (prec == STAP_PREC_FP32) hipLaunchKernelGGL((inner_batched_kernel<ST, DP, 4, true>), g, block, 0, st, desc, n);
        else hipLaunchKernelGGL((inner_batched_kernel<ST, DP, 4, false>), g, block, 0, st, desc, n);
      }
      return hipGetLastError();
    });
  });
}

hipError_t launch_inner(const Dims& d, const float2* w, const float2* snap, float* power, float2* y,
                        hipStream_t st) {
  const dim3 g(d.P * d.B);
  if (d.prec == STAP_PREC_FP32 && f32_form(d.D, d.S, d.N))
    return by_f32(d.D, d.S, [&](auto sc, auto dc) {
      hipLaunchKernelGGL((inner_f32_kernel<sc.value, dc.value>), g, dim3(256), 0, st, w, snap, power, y, d);
      return hipGetLastError();
    });
  return by_steer(d.S, [&](auto sc) {
    return by_dof(d.D, [&](auto dc) -> hipError_t {
      constexpr int ST = sc.value, DP = dc.value;
      // the wave counts that waves_of() gives for this shape at any block length
      auto go = [&](auto nw) {
        constexpr int NW = nw.value;
        if constexpr (NW == 4 || NW == waves_of(ST, DP, 16) || NW == waves_of(ST, DP, 32) || NW == waves_of(ST, DP, 65)) {
          if (DP > 128 || d.prec == STAP_PREC_FP32)
            hipLaunchKernelGGL((inner_kernel<ST, DP, NW, true>), g, dim3(64 * NW), 0, st, w, snap, power, y, d);
          else
            hipLaunchKernelGGL((inner_kernel<ST, DP, NW, DP >= 192>), g, dim3(64 * NW), 0, st, w, snap, power, y, d);
        }
        return hipGetLastError();
      };
      switch (waves_of(ST, DP, d.N)) {
        case 1: return go(std::integral_constant<int, 1>{});
        case 2: return go(std::integral_constant<int, 2>{});
        case 8: return go(std::integral_constant<int, 8>{});
      }
      return go(std::integral_constant<int, 4>{});
    });
  });
}

}  // namespace stap
