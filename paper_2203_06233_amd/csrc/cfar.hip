// Cell-averaging CFAR detection along range on the AMF power map
// power[P][S][R] (the textbook CA-CFAR detector applied to the output of the
// STAP chain; not part of the paper's kernel, which ends at the output
// power).  For cell r of a row the reference cells are n_ref cells on each
// side beyond n_guard guard cells; cells outside [0, R) are left out and
// n_used counts the rest.  Detection: power[r] * n_used > alpha * sum.
//
// The decision is an integer result of floating-point arithmetic, so its
// arithmetic is fixed: the reference cells are added in FP64, one at a time,
// in increasing offset order (left window, then right window, a missing
// cell adding 0), and the test is taken in FP64 with no fused multiply-add.
// Any implementation that keeps this order returns the same mask bit for bit.
//
// The ordered sum itself is needed only where it decides: the FP32 sum of
// the same cells in any order is within a few hundred FP32 roundings of it
// (the cells are not negative), so a cell whose two sides differ by more than
// kMargin of the threshold side is settled by whatever sum is cheap, and the
// ordered FP64 sums are formed only by threads that hold a cell inside the
// margin, or any value that is negative or not finite.
//
// One workgroup takes kTile cells of one (bin, steering) row plus a halo of
// n_guard + n_ref cells per side.  Each thread owns kRun consecutive cells,
// whose windows share all but the outer kRun - 1 values on either end: suffix
// sums of the first kRun - 1 values, the shared middle, prefix sums of the
// last, two additions per cell (37 instead of 128 per side with 16 reference
// cells).  The cells are staged twice in LDS, once so that the threads' left
// windows start at kRun times the thread index and once for the right ones,
// with a pad word every kRun: a window's m-th value then sits at a constant
// distance from the thread's base (no address arithmetic per read) and the
// lanes' reads fall in distinct banks.  (Four pad words and 16-byte reads take
// half as much LDS again, two workgroups fewer per CU: 315 us against 261.)
// A tile's loads are issued together, at clamped addresses: behind a bounds
// check each is waited for by itself (250 us with that, all else as here).
// 256 x 32 x 16384 cells with 16 reference cells a side: 334 us with the
// ordered sums throughout, 161 so (4.2 TB/s of 4 bytes in and 1 out per
// cell); what is left is arithmetic that overlaps the loads of other
// workgroups only in part.
#include "common.h"
#include "kernels.h"

namespace stap {

namespace {

constexpr int kRun = 8;                   // consecutive cells per thread
constexpr int kThreads = 256;
constexpr int kTile = kRun * kThreads;    // cells per workgroup
constexpr int lds_index(int i) { return i + (i >> 3); }
// left copy: cells from t0 - H on, up to the tile's last cell; right copy:
// cells from t0 + n_guard + 1 on; both with the ordered sums' look-ahead
constexpr int kLeftWords = lds_index(kTile + kMaxCfarRef + kMaxCfarGuard + kRun) + 1;
constexpr int kRightWords = lds_index(kTile + kMaxCfarRef + kRun) + 1;
// above 8 (kMaxCfarRef + 2 kRun) FP32 roundings
constexpr float kMargin = 0x1p-13f;

// Sum of n window values in order for each of the thread's kRun cells: cell j
// adds w[j], w[j+1], ..., w[j+n-1] with w[m] at LDS index base + m.
__device__ __forceinline__ void window_sums(const float* s, int base, int n, double (&acc)[kRun]) {
  double ring[kRun];
#pragma unroll
  for (int m = 0; m < kRun; ++m) ring[m] = (double)s[lds_index(base + m)];
  for (int i0 = 0; i0 < n; i0 += kRun) {
#pragma unroll
    for (int u = 0; u < kRun; ++u) {
      if (i0 + u < n) {
        // step i = i0 + u: ring slot (i + j) % kRun holds w[i + j]
#pragma unroll
        for (int j = 0; j < kRun; ++j) acc[j] += ring[(u + j) % kRun];
        ring[u] = (double)s[lds_index(base + i0 + u + kRun)];
      }
    }
  }
}

// The same sums in any order and in FP32, n >= kRun, w[m] at a[lds_index(m)]
// (a the thread's base).
__device__ __forceinline__ void window_sums_any(const float* a, int n, float (&acc)[kRun]) {
  float suf[kRun];
  suf[kRun - 1] = 0.f;
#pragma unroll
  for (int m = kRun - 2; m >= 0; --m) suf[m] = suf[m + 1] + a[m];
  float mid = a[kRun - 1];
  const float* p = a + kRun + 1;
  int m = kRun;
  for (; m + kRun <= n; m += kRun, p += kRun + 1)
    mid += ((p[0] + p[1]) + (p[2] + p[3])) + ((p[4] + p[5]) + (p[6] + p[7]));
  for (int i = 0; m + i < n; ++i) mid += p[i];
#pragma unroll
  for (int j = 0; j < kRun; ++j) {
    acc[j] += suf[j] + mid;
    if (j + 1 < kRun) mid += a[lds_index(n + j)];
  }
}

__global__ __launch_bounds__(kThreads) void cfar_kernel(const float* __restrict__ power,
                                                        unsigned char* __restrict__ detect, int R, int tiles_per_row,
                                                        int n_ref, int n_guard, double alpha) {
#pragma clang fp contract(off)
  __shared__ float sl[kLeftWords], sr[kRightWords];
  __shared__ int negative[kThreads / 64];
  const int row = blockIdx.x / tiles_per_row;
  const int tile = blockIdx.x - row * tiles_per_row;
  const int t0 = tile * kTile;          // first cell of the tile
  const int H = n_ref + n_guard;        // halo per side
  const float* prow = power + (long long)row * R;
  // stage cells t0 - H .. t0 + kTile + H - 1 (zero outside the row), plus
  // kRun values of look-ahead (read, but in no sum)
  const int nl = kTile + H + kRun, off = H + n_guard + 1, span = kTile + 2 * H;
  const bool inside = t0 >= H && t0 + kTile + H <= R;
  // staged value i is cell t0 - H + i; first and last of them in the row
  const float* const p0 = prow + (t0 - H);
  const int first = max(H - t0, 0), last = min(span, R - t0 + H) - 1;
  unsigned int sign = 0;  // the sign bit is set if any value has it
  float v[kRun + 1];      // the tile's loads at once: none behind a branch
#pragma unroll
  for (int u = 0; u <= kRun; ++u) v[u] = p0[(unsigned)min(max((int)threadIdx.x + u * kThreads, first), last)];
#pragma unroll
  for (int u = 0; u <= kRun; ++u) asm volatile("" : "+v"(v[u]));
  if (!inside) {
#pragma unroll
    for (int u = 0; u <= kRun; ++u) {
      const int i = threadIdx.x + u * kThreads;
      if (i < first || i > last) v[u] = 0.f;
    }
  }
#pragma unroll
  for (int u = 0; u <= kRun; ++u) sign |= __float_as_uint(v[u]);
  // lds_index(i + u kThreads) = lds_index(i) + u kStep; from u = 1 on every
  // value belongs to both copies, up to the tile's last cell to the left one
  constexpr int kStep = lds_index(kThreads);
  static_assert(kThreads % 8 == 0 && kThreads > 2 * kMaxCfarGuard + kMaxCfarRef, "");
  float* const pl = sl + lds_index(threadIdx.x);
  const int ir = lds_index((int)threadIdx.x - off);
  if ((int)threadIdx.x >= off) sr[ir] = v[0];
#pragma unroll
  for (int u = 0; u < kRun; ++u) {
    pl[u * kStep] = v[u];
    if (u > 0) sr[ir + u * kStep] = v[u];
  }
  for (int i = threadIdx.x + kTile; i < span + kRun; i += kThreads) {
    const float x = i < kTile + kThreads ? v[kRun] : i <= last ? p0[i] : 0.f;
    sign |= __float_as_uint(x);
    if (i < nl) sl[lds_index(i)] = x;
    sr[lds_index(i - off)] = x;
  }
  const bool neg = __any(sign >> 31);
  if ((threadIdx.x & 63) == 0) negative[threadIdx.x >> 6] = neg;
  __syncthreads();

  const int base = kRun * threadIdx.x, c0 = t0 + base;  // the thread's first cell
  if (c0 >= R) return;
  // Reference cells of cell j that exist: left [c-g-n, c-g-1] and right
  // [c+g+1, c+g+n]; all of them away from the ends of the row.
  auto used = [&](int j) {
    if (inside) return 2 * n_ref;
    const int c = c0 + j;
    const int l_lo = max(c - n_guard - n_ref, 0), l_hi = min(c - n_guard - 1, R - 1);
    const int r_lo = max(c + n_guard + 1, 0), r_hi = min(c + n_guard + n_ref, R - 1);
    return max(l_hi - l_lo + 1, 0) + max(r_hi - r_lo + 1, 0);
  };
  unsigned int lo = 0, hi = 0;  // the mask bytes of cells 0-3 and 4-7
  auto put = [&](int j, bool hit) {
    const unsigned int b = hit ? 1u << (8 * (j & 3)) : 0u;
    if (j < 4) lo |= b;
    else hi |= b;
  };
  const float al = (float)alpha;
  bool settled = n_ref >= kRun && al > 0x1p-60f && al < 0x1p60f;
#pragma unroll
  for (int w = 0; w < kThreads / 64; ++w) settled = settled && !negative[w];
  if (settled) {
    float acc[kRun], top = 0.f;
#pragma unroll
    for (int j = 0; j < kRun; ++j) acc[j] = 0.f;
    window_sums_any(sl + lds_index(base), n_ref, acc);
    window_sums_any(sr + lds_index(base), n_ref, acc);
    // A cell is settled if its distance from the threshold exceeds the margin
    // (2^-100 more where products lose bits): false for a NaN on either side
    // and for an infinite sum.  An infinite threshold product is above any
    // cell below 2^120.  A zero sum of values that are not negative is zero
    // in any order.
    const float almargin = al * kMargin;
    bool clear = true, clear_or_zero = true;
#pragma unroll
    for (int j = 0; j < kRun; ++j) {
      const float p = sl[lds_index(base + H + j)];
      const float gap = fmaf(-al, acc[j], p * (float)used(j));
      const bool ok = fabsf(gap) > fmaf(almargin, acc[j], 0x1p-100f);
      top = fmaxf(top, p);
      clear = clear && ok;
      clear_or_zero = clear_or_zero && (ok || acc[j] == 0.f);
      put(j, gap > 0.f);
    }
    settled = top < 0x1p120f && (clear || clear_or_zero);
  }
  if (!settled) {
    lo = hi = 0;
    double acc[kRun];
#pragma unroll
    for (int j = 0; j < kRun; ++j) acc[j] = 0.0;
    window_sums(sl, base, n_ref, acc);  // offsets -(g+n) .. -(g+1)
    window_sums(sr, base, n_ref, acc);  // offsets g+1 .. g+n
#pragma unroll
    for (int j = 0; j < kRun; ++j)
      put(j, (double)sl[lds_index(base + H + j)] * (double)used(j) > alpha * acc[j]);
  }
  const unsigned long long bits = ((unsigned long long)hi << 32) | lo;
  unsigned char* out = detect + (long long)row * R + c0;
  if (c0 + kRun <= R && ((reinterpret_cast<uintptr_t>(out) & 7) == 0)) {
    *reinterpret_cast<unsigned long long*>(out) = bits;
  } else {
#pragma unroll
    for (int j = 0; j < kRun; ++j)
      if (c0 + j < R) out[j] = (unsigned char)((bits >> (8 * j)) & 1u);
  }
}

}  // namespace

hipError_t launch_cfar(const Dims& d, int n_ref, int n_guard, double alpha, const float* power,
                       unsigned char* detect, hipStream_t st) {
  const int tiles = (d.R + kTile - 1) / kTile;
  const long long rows = (long long)d.P * d.S;
  if (rows * tiles > 0x7fffffffLL) return hipErrorInvalidValue;
  hipLaunchKernelGGL(cfar_kernel, dim3((unsigned)(rows * tiles)), dim3(kThreads), 0, st, power, detect, d.R, tiles,
                     n_ref, n_guard, alpha);
  return hipGetLastError();
}

}  // namespace stap
