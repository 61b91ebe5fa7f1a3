// Doppler filtering with time-staggered DOF (statements S and T of the STAP
// kernel, Sec. 4.2; Table 2 row fft_{2D,axis=1}).
//
//   X[k][t*C+c][r] = sum_p h[p-t] x[c][p][r] exp(-2 pi i k p / P)
//
// or, with each tap referenced to its own first pulse (relative phase),
// exp(-2 pi i k (p - t) / P), i.e. the absolute form times exp(2 pi i k t / P).
//
// One workgroup takes one channel c and RT consecutive range cells.  The
// length-P DFT is split as P = P1 * P2 (p = P2*n1 + n2, k = k1 + P1*k2):
//   pass 1  each thread owns one (n2, cell) and keeps the P1 samples
//           x[P2*n1 + n2], n1 = 0..P1-1, in registers (loaded once, coalesced
//           along range), windows them for tap t, runs a P1-point DFT in
//           registers and multiplies by exp(-2 pi i k1 n2 / P);
//   LDS     one transpose through a [k1][n2][cell] tile;
//   pass 2  each (k1, cell) runs a P2-point DFT in registers and stores bins
//           k1 + P1*k2 straight to X[k][d][r] (range fastest, coalesced).
// The cube is read from HBM once for all T taps; with subarrays, each
// channel's samples are the sum of its elements, formed as they are loaded.
// P = 100 (the paper's pulse count) runs the same passes as 10 x 10 with
// direct in-register DFTs.  Twiddles of the inner DFTs
// are compile-time constants; the P-point twiddles and the Hann window come
// from correctly rounded compile-time tables, staged once per workgroup in LDS.
//
// The pass is bound by HBM, and how close it comes is set by the length of
// the runs it touches (RT cells of 8 bytes in each of P rows read and P T
// rows written) and by the waves in flight.  Copies of the same access
// pattern without the arithmetic reach 4.6 TB/s with 128-byte runs and 5.0
// with 256-byte ones on the 32 x 256 x 16384 cube.  Every pulse count
// therefore has a narrow tile (256 threads) and, where the registers allow
// it, a wide one that needs enough cells to fill the chip:
//                                             before    narrow     wide
//    32 pulses, 32 channels, 16384 cells      0.101     0.100             ms
//    64 pulses, 64 channels,  4096 cells      0.096     0.102    0.095
//   128 pulses, 16 channels,  4096 cells      0.056      0.055    0.050
//   256 pulses, 32 channels, 16384 cells      0.94       0.94     0.86
//   512 pulses, 64 channels,  4096 cells      1.45       1.01     0.90
//   100 pulses, 1000 elements, 30000 cells    5.03       5.0      4.08
// (before: the narrow tile with the subarray loads in every kernel).
#include <type_traits>

#include "common.h"
#include "kernels.h"

namespace stap {

// P = P1 * P2; RT range cells and NT threads per workgroup; WPE waves per
// SIMD the registers are held to.  WIDE: the tile for large launches.
template <int P, bool WIDE>
struct FftShape {
  static constexpr int LOG = ilog2(P);
  static constexpr int P1 = 1 << ((LOG + 1) / 2);
  static constexpr int P2 = P / P1;
  static constexpr int RT = !WIDE ? 256 / P2 : P == 64 ? 128 : P == 128 ? 64 : P >= 256 ? 32 : 256 / P2;
  static constexpr int NT = P2 * RT;
  static constexpr int WPE = P == 512 ? 1 : P == 256 && !WIDE ? 3 : 4;
  // Elements loaded at a time (subarrays): four where a thread has eight
  // samples of each, so that enough loads are in flight (32 pulses, 6 channels
  // of 25 elements x 2000 cells: 19.2 us with one, 13.8 with four; 64 pulses,
  // 6 of 10 x 6154: 52.6 and 50.0).  From 128 pulses on one fills the registers.
  static constexpr int ELEMS = !WIDE && P <= 64 ? 4 : 1;
  // Whether the compiler is kept from gathering all window, twiddle and
  // address values of an unrolled loop before their use: only where the
  // registers need it (256 pulses, narrow, 8 channels x 1024 cells: 12.4 us
  // with it, 11.3 without).
  static constexpr bool FENCE = WIDE || P == 512;
  // Complex values of the transpose tile.  Narrow tiles of up to 64 pulses take
  // 40 KB of LDS, which holds a compute unit to four workgroups: with the six
  // to eight that their registers allow, more rows are open in memory at a time
  // (32 pulses, 32 channels x 16384 cells, T = 3: 105 us, so 100).
  static constexpr int TILE = !WIDE && P <= 64 ? 4900 : P1 * P2 * RT;
};
// The paper's 100 pulses: 10 x 10, 32 or 96 cells (whole 128-byte lines).
// With subarrays the loads of several elements are issued before their
// additions so that enough of them are in flight to stream the cube; the
// wide tile, with three times the waves per workgroup, needs fewer.
template <bool WIDE>
struct FftShape<100, WIDE> {
  static constexpr int P1 = 10, P2 = 10, RT = WIDE ? 96 : 32, NT = 10 * RT, WPE = 4, ELEMS = WIDE ? 2 : 4;
  static constexpr bool FENCE = WIDE;
  static constexpr int TILE = 100 * RT;
};

// One workgroup's tile: channel c, range cells r0 .. r0+RT-1 of one cube.
// SUB: the subarray loads are compiled in (with d.sub == 1 they are not used).
template <int P, bool WIDE, bool SUB>
__device__ __forceinline__ void doppler_tile(const float2* __restrict__ cube, float2* __restrict__ snap,
                                             const Dims& d, int c, int r0) {
  using Sh = FftShape<P, WIDE>;
  constexpr int P1 = Sh::P1, P2 = Sh::P2, RT = Sh::RT, NT = Sh::NT;
  __shared__ float2 ybuf[Sh::TILE];  // [k1][n2][cell]
  __shared__ float2 tw[P];
  __shared__ float hwin[P];

  const int tid = threadIdx.x;

  for (int m = tid; m < P; m += NT) {
    tw[m] = make_float2(kTwTab<P>.c[m], -kTwTab<P>.s[m]);
    hwin[m] = kWinTab<P>.h[d.T - 1][m];
  }

  const int col = tid % RT, n2 = tid / RT;
  const int r = r0 + col;
  const bool live = r < d.R;
  float2 x[P1];
#pragma unroll
  for (int n1 = 0; n1 < P1; ++n1) x[n1] = make_float2(0.f, 0.f);
  if (live && (!SUB || d.sub == 1)) {
    const float2* src = cube + (long long)c * d.sc + (long long)n2 * d.sp + r;
#pragma unroll
    for (int n1 = 0; n1 < P1; ++n1) {
      x[n1] = load_stream(src + (long long)(P2 * n1) * d.sp);
      if (Sh::FENCE && n1 % 8 == 7) __builtin_amdgcn_sched_barrier(0);
    }
  } else if (live) {
    // channel c is the sum of array elements c*sub .. c*sub + sub - 1,
    // added in element order
    constexpr int EU = Sh::ELEMS;
    int e = 0;
    for (; e + EU <= d.sub; e += EU) {
      float2 v[EU][P1];
#pragma unroll
      for (int u = 0; u < EU; ++u) {
        const float2* src = cube + (long long)(c * d.sub + e + u) * d.sc + r;
#pragma unroll
        for (int n1 = 0; n1 < P1; ++n1) v[u][n1] = load_stream(src + (long long)(P2 * n1 + n2) * d.sp);
      }
#pragma unroll
      for (int u = 0; u < EU; ++u)
#pragma unroll
        for (int n1 = 0; n1 < P1; ++n1) {
          x[n1].x += v[u][n1].x;
          x[n1].y += v[u][n1].y;
        }
    }
    for (; e < d.sub; ++e) {
      const float2* src = cube + (long long)(c * d.sub + e) * d.sc + r;
#pragma unroll
      for (int n1 = 0; n1 < P1; ++n1) {
        const float2 v = load_stream(src + (long long)(P2 * n1 + n2) * d.sp);
        x[n1].x += v.x;
        x[n1].y += v.y;
      }
    }
  }
  __syncthreads();

  for (int t = 0; t < d.T; ++t) {
    float2 v[P1];
#pragma unroll
    for (int n1 = 0; n1 < P1; ++n1) {
      const int q = P2 * n1 + n2 - t;
      const float h = (q >= 0 && q < P) ? hwin[q] : 0.f;
      v[n1] = make_float2(x[n1].x * h, x[n1].y * h);
      if (Sh::FENCE && n1 % 8 == 7) __builtin_amdgcn_sched_barrier(0);
    }
    dft_any<P1>(v);
#pragma unroll
    for (int k1 = 0; k1 < P1; ++k1) {
      const float2 y = (k1 == 0) ? v[k1] : cmul(v[k1], tw[k1 * n2]);
      ybuf[(k1 * P2 + n2) * RT + col] = y;
      if (Sh::FENCE && k1 % 4 == 3) __builtin_amdgcn_sched_barrier(0);
    }
    __syncthreads();
    const int dof = t * d.C + c;
    for (int task = tid; task < P1 * RT; task += NT) {
      const int c3 = task % RT, k1 = task / RT;
      float2 z[P2];
#pragma unroll
      for (int m2 = 0; m2 < P2; ++m2) z[m2] = ybuf[(k1 * P2 + m2) * RT + c3];
      dft_any<P2>(z);
      const int r3 = r0 + c3;
      if (d.tap_rel && t > 0) {
        // tap t referenced to its own first pulse: times exp(+2 pi i k t / P)
#pragma unroll
        for (int k2 = 0; k2 < P2; ++k2) {
          z[k2] = cmulc(z[k2], tw[((k1 + P1 * k2) * t) % P]);
          if (Sh::FENCE && k2 % 4 == 3) __builtin_amdgcn_sched_barrier(0);
        }
      }
      if (r3 < d.R) {
        float2* dst = snap + ((long long)k1 * d.D + dof) * d.R + r3;
        const long long step = (long long)P1 * d.D * d.R;
#pragma unroll
        for (int k2 = 0; k2 < P2; ++k2) {
          store_stream(dst, z[k2]);
          dst += step;
          if (Sh::FENCE && k2 % 4 == 3) __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
    __syncthreads();
  }
}

// Tile of a workgroup.  Workgroups go round-robin over the eight XCDs; with
// long transforms each XCD takes one contiguous part of the tiles instead,
// so that neighbouring runs of a row are written through the same L2 at about
// the same time (0.88 -> 0.86 ms on the 32 x 256 x 16384 cube; with up to
// 128 pulses the plain order is as fast or faster).
template <int P, bool WIDE>
constexpr bool kByXcd = WIDE && P >= 256;
template <int P, bool WIDE>
__device__ __forceinline__ int tile_of(int id, int n) {
  if (!kByXcd<P, WIDE>) return id;
  const int xcd = id & 7;
  return xcd * (n >> 3) + min(xcd, n & 7) + (id >> 3);
}

template <int P, bool WIDE, bool SUB>
__global__ __launch_bounds__((FftShape<P, WIDE>::NT)) __attribute__((amdgpu_waves_per_eu(FftShape<P, WIDE>::WPE)))
void doppler_kernel(const float2* __restrict__ cube, float2* __restrict__ snap, Dims d) {
  constexpr int RT = FftShape<P, WIDE>::RT;
  if constexpr (kByXcd<P, WIDE>) {
    const int ntr = (d.R + RT - 1) / RT;
    const int u = tile_of<P, WIDE>(blockIdx.x, gridDim.x);
    doppler_tile<P, WIDE, SUB>(cube, snap, d, u / ntr, (u % ntr) * RT);
  } else {  // a grid of tiles x channels: no division
    doppler_tile<P, WIDE, SUB>(cube, snap, d, blockIdx.y, blockIdx.x * RT);
  }
}

// Batched: the workgroups of several cubes with the same P in one grid.
template <int P, bool WIDE, bool SUB>
__global__ __launch_bounds__((FftShape<P, WIDE>::NT)) __attribute__((amdgpu_waves_per_eu(FftShape<P, WIDE>::WPE)))
void doppler_batched_kernel(const ProbDesc* __restrict__ desc, BatchIndex bi) {
  constexpr int RT = FftShape<P, WIDE>::RT;
  const int g = tile_of<P, WIDE>(blockIdx.x, gridDim.x);
  int j = 0;
  while (j + 1 < bi.n && bi.tile_begin[j + 1] <= g) ++j;
  const ProbDesc& pd = desc[bi.prob[j]];
  const Dims d = pd.d;
  const int local = g - bi.tile_begin[j];
  const int ntr = (d.R + RT - 1) / RT;
  doppler_tile<P, WIDE, SUB>(pd.cube, pd.snap, d, local / ntr, (local % ntr) * RT);
}

namespace {

template <class F>
auto by_pulse(int P, F&& f) {
  switch (P) {
    case 32: return f(std::integral_constant<int, 32>{});
    case 64: return f(std::integral_constant<int, 64>{});
    case 100: return f(std::integral_constant<int, 100>{});
    case 128: return f(std::integral_constant<int, 128>{});
    case 256: return f(std::integral_constant<int, 256>{});
  }
  return f(std::integral_constant<int, 512>{});
}

}  // namespace

int doppler_tiles(const Dims& d, bool wide) {
  return by_pulse(d.P, [&](auto p) {
    const int rt = wide ? FftShape<p.value, true>::RT : FftShape<p.value, false>::RT;
    return (d.R + rt - 1) / rt * d.C;
  });
}

// Wide tiles where their workgroups give every compute unit 16 waves; with
// subarrays only the 100-pulse shape has one.  With a single tap a tile's
// loads and stores take equally long, and a compute unit that holds one wide
// workgroup does them in turn: at 64, 100, 256 and 512 pulses narrow tiles are
// as fast or faster then (32 channels, 4096 cells: 23, 44, 100 and 214 us
// against 28, 47, 108 and 236), at 128 not (48 against 46), and at 100 not
// where many elements a subarray make the loads long (20 channels x 3000
// cells of 10 elements: 115 against 100 us; 8 x 4096 of 4: 26 against 28).
bool doppler_wide(int P, int sub, bool one_tap, long long wide_tiles) {
  if (P == 32 || (sub > 1 && P != 100) || (one_tap && P != 128 && !(P == 100 && sub >= 8))) return false;
  return by_pulse(P, [&](auto p) { return wide_tiles * FftShape<p.value, true>::NT >= 256LL * 1024; });
}

// The narrow kernel without subarrays.  At 100 pulses it is the one that has
// their loads too: its registers are allocated better (one tap, 32 channels x
// 4096 cells 44 us, without those loads 47).
template <int P>
constexpr bool kPlainSub = P == 100;

hipError_t launch_doppler_batched(int P, const ProbDesc* desc, const BatchIndex& bi, int tiles, bool wide, bool sub,
                                  hipStream_t st) {
  if (tiles <= 0) return hipSuccess;
  return by_pulse(P, [&](auto p) {
    constexpr int Q = p.value;
    constexpr bool W = Q != 32, WS = Q == 100;
    const dim3 g(tiles), wt(FftShape<Q, W>::NT), nt(FftShape<Q, false>::NT);
    if (!sub && wide) hipLaunchKernelGGL((doppler_batched_kernel<Q, W, false>), g, wt, 0, st, desc, bi);
    else if (!sub) hipLaunchKernelGGL((doppler_batched_kernel<Q, false, kPlainSub<Q>>), g, nt, 0, st, desc, bi);
    else if (WS && wide) hipLaunchKernelGGL((doppler_batched_kernel<Q, WS, true>), g, wt, 0, st, desc, bi);
    else hipLaunchKernelGGL((doppler_batched_kernel<Q, false, true>), g, nt, 0, st, desc, bi);
    return hipGetLastError();
  });
}

hipError_t launch_doppler(const Dims& d, const float2* cube, float2* snap, hipStream_t st) {
  const bool sub = d.sub > 1, wide = doppler_wide(d.P, d.sub, d.T == 1, doppler_tiles(d, true));
  return by_pulse(d.P, [&](auto p) {
    constexpr int Q = p.value;
    constexpr bool W = Q != 32, WS = Q == 100;
    const int tiles = doppler_tiles(d, wide);
    const dim3 g = wide && kByXcd<Q, true> ? dim3(tiles) : dim3(tiles / d.C, d.C);
    const dim3 wt(FftShape<Q, W>::NT), nt(FftShape<Q, false>::NT);
    if (!sub && wide) hipLaunchKernelGGL((doppler_kernel<Q, W, false>), g, wt, 0, st, cube, snap, d);
    else if (!sub) hipLaunchKernelGGL((doppler_kernel<Q, false, kPlainSub<Q>>), g, nt, 0, st, cube, snap, d);
    else if (WS && wide) hipLaunchKernelGGL((doppler_kernel<Q, WS, true>), g, wt, 0, st, cube, snap, d);
    else hipLaunchKernelGGL((doppler_kernel<Q, false, true>), g, nt, 0, st, cube, snap, d);
    return hipGetLastError();
  });
}

}  // namespace stap
