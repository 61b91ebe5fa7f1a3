// Stage weight solve on the matrix cores: one workgroup per system reads the
// loaded covariance from global memory and runs bsolve_blocks()
// (bsolve_impl.h), with or without FP64 refinement.
#include "bsolve_impl.h"
#include "kernels.h"

namespace stap {

namespace {

// R_L in global memory, of which the lower triangle is read.
struct GlobalRB {
  const float2* A;
  int D;
  bool vec;  // rows16(A, D)
  // Lane (m, q): R[16I + m][16J + 4q + i], i = 0..3 (J <= I), identity beyond
  // D; the diagonal's imaginary part is not looked at.
  __device__ __forceinline__ Acc block(int I, int J) const {
    const int l = lane_tid() & 63, m = l & 15, q = l >> 4;
    const int r = 16 * I + m, c0 = 16 * J + 4 * q;
    Acc a;
    float2 v[4];
    if (J < I) {
      load4(A, r, c0, r < D, D, vec, v);
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int c = c0 + i;
        v[i] = make_float2(r == c ? 1.f : 0.f, 0.f);
        if (r < D && c < D) {
          v[i] = c <= r ? A[r * D + c] : A[c * D + r];
          v[i].y = c > r ? -v[i].y : c == r ? 0.f : v[i].y;
        }
      }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      a.re[i] = v[i].x;
      a.im[i] = v[i].y;
    }
    return a;
  }
  __device__ __forceinline__ Acc get(int J, int I, int) const {
    if (J <= I) {  // conj(R[16I + m][16J + 4q + s])
      Acc a = block(I, J);
      a.im = -a.im;
      return a;
    }
    const int l = lane_tid() & 63, m = l & 15, q = l >> 4;
    Acc a;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = 16 * J + 4 * q + i, c = 16 * I + m;
      const float2 v = (r < D && c < D) ? A[r * D + c] : make_float2(0.f, 0.f);
      a.re[i] = v.x;
      a.im[i] = v.y;
    }
    return a;
  }
};

// With refinement and 8 waves the register allocation is capped at 128 so
// that two systems share a compute unit (no more than 4 registers spill with
// up to 3 L and 2 M slots, 26 to 170 with more).
template <int NSL, int NSM, int NW, int LEVEL>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(LEVEL != kPlain && NW == 8 ? 4 : 1)))
void bsolve_kernel(const float2* __restrict__ cov,
                                                         const float2* __restrict__ steer,
                                                         float2* __restrict__ wout, int* __restrict__ info_out,
                                                         Dims d) {
  using C = BCfg<NSL, NSM, NW>;
  extern __shared__ __align__(16) unsigned char lds[];
  const int sys = blockIdx.x;
  const float2* const A = cov + (long long)sys * d.D * d.D;
  const float2* const V = steer + steer_offset(d, sys);
  const GlobalRB R{A, d.D, rows16(A, d.D)};
  const Slots<C> sl(d.D, d.S, __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6));
  const SolveLds<C, LEVEL> L(lds, sl.NB, sl.NS);
  const int m = lane_tid() & 15, q = (lane_tid() & 63) >> 4;
  Acc al[NSL], am[NSM];
  float top = 0.f;  // with refinement: the lane's largest of every 64th diagonal element
  if (LEVEL != kPlain)
    for (int r = threadIdx.x & 63; r < d.D; r += 64) top = fmaxf(top, A[r * (d.D + 1)].x);
#pragma unroll
  for (int t = 0; t < NSL; ++t) {
    al[t] = acc_zero();
    if (sl.lv[t]) {
      al[t] = R.block(sl.lr[t], sl.lc[t]);
      if (sl.lr[t] == sl.lc[t]) {
        const float rd = blk_diag(al[t]);
        if (m >> 2 == q) L.rdiag[16 * sl.lr[t] + m] = rd;
      }
      al[t] = acc_neg(al[t]);
    }
  }
  load_steer(sl, V, d.D, d.S, am);
  for (int r = threadIdx.x; r < 16 * sl.NB; r += C::NT) L.d64[r] = 0.0;
  for (int o = 32; o > 0; o >>= 1) top = fmaxf(top, __shfl_xor(top, o));
  const SysScale sc(top);
  if (LEVEL != kPlain) {
#pragma unroll
    for (int t = 0; t < NSL; ++t) al[t] = acc_scale(al[t], sc.r);  // the identity beyond D scales with the rest
  }
  bsolve_blocks<C, LEVEL>(sl, al, am, L, R, V, wout + (long long)sys * d.S * d.D, info_out ? info_out + sys : nullptr,
                          d, nullptr, sc);
}

template <int NSL, int NSM, int NW, int LEVEL>
hipError_t go_r(const Dims& d, const float2* cov, const float2* steer, float2* w, int* info, hipStream_t st) {
  const size_t lds = BCfg<NSL, NSM, NW>::lds_bytes((d.D + 15) / 16, (d.S + 15) / 16, LEVEL);
  if (lds > 48 * 1024) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&bsolve_kernel<NSL, NSM, NW, LEVEL>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL((bsolve_kernel<NSL, NSM, NW, LEVEL>), dim3(d.P * d.B), dim3(64 * NW), lds, st, cov, steer, w,
                     info, d);
  return hipGetLastError();
}

template <int NSL, int NSM, int NW>
hipError_t go(const Dims& d, const float2* cov, const float2* steer, float2* w, int* info, hipStream_t st) {
  if (d.refine == 0) return go_r<NSL, NSM, NW, kPlain>(d, cov, steer, w, info, st);
  if constexpr (NW != 4)  // four waves run where they were asked for, the corrected form where nothing was
    if (d.corr) return go_r<NSL, NSM, NW, kCorrected>(d, cov, steer, w, info, st);
  return go_r<NSL, NSM, NW, kRefined>(d, cov, steer, w, info, st);
}

template <int NW>
int round_up(int need, const int* opts, int n) {
  for (int i = 0; i < n; ++i)
    if (need <= opts[i]) return opts[i];
  return 0;
}

}  // namespace

// Slot counts instantiated per wave count: L slots {1, 2, 3, 5} (4 waves),
// {2, 3, 5} (8 waves) or {3, 5} (16 waves), M slots {1, 2, 4} ({2, 3} with
// 16 waves).  Variant 8 runs D > 128 (up to 12 block columns) with 16 waves.
static const int kL4[] = {1, 2, 3, 5}, kL8[] = {2, 3, 5}, kL16[] = {3, 5}, kM[] = {1, 2, 4}, kM16[] = {2, 3};

static int waves_for(const Dims& d, int waves) { return waves == 8 && d.D > 128 ? 16 : waves; }

static bool slots_for(const Dims& d, int waves, int& nl, int& nm) {
  const int NB = (d.D + 15) / 16, NS = (d.S + 15) / 16;
  if (waves == 4) {
    nl = round_up<4>(BCfg<1, 1, 4>::lslots(NB), kL4, 4);
    nm = round_up<4>(BCfg<1, 1, 4>::mslots(NB, NS), kM, 3);
  } else if (waves == 8) {
    nl = round_up<8>(BCfg<1, 1, 8>::lslots(NB), kL8, 3);
    nm = round_up<8>(BCfg<1, 1, 8>::mslots(NB, NS), kM, 3);
  } else if (waves == 16) {
    nl = round_up<16>(BCfg<1, 1, 16>::lslots(NB), kL16, 2);
    nm = round_up<16>(BCfg<1, 1, 16>::mslots(NB, NS), kM16, 2);
  } else {
    return false;
  }
  return nl > 0 && nm > 0;
}

bool bsolve_supported(const Dims& d, int waves) {
  int nl, nm;
  return d.D <= kMaxDof && slots_for(d, waves_for(d, waves), nl, nm);
}

hipError_t launch_bsolve(const Dims& d, const float2* cov, const float2* steer, float2* w, int* info,
                         hipStream_t st, int waves_asked) {
  int nl, nm;
  const int waves = waves_for(d, waves_asked);
  if (!slots_for(d, waves, nl, nm)) return hipErrorInvalidValue;
#define STAP_BS(L, M, W) \
  if (nl == L && nm == M && waves == W) return go<L, M, W>(d, cov, steer, w, info, st);
  STAP_BS(1, 1, 4) STAP_BS(1, 2, 4) STAP_BS(1, 4, 4)
  STAP_BS(2, 1, 4) STAP_BS(2, 2, 4) STAP_BS(2, 4, 4)
  STAP_BS(3, 1, 4) STAP_BS(3, 2, 4) STAP_BS(3, 4, 4)
  STAP_BS(5, 1, 4) STAP_BS(5, 2, 4) STAP_BS(5, 4, 4)
  STAP_BS(2, 1, 8) STAP_BS(2, 2, 8) STAP_BS(2, 4, 8)
  STAP_BS(3, 1, 8) STAP_BS(3, 2, 8) STAP_BS(3, 4, 8)
  STAP_BS(5, 1, 8) STAP_BS(5, 2, 8) STAP_BS(5, 4, 8)
  STAP_BS(3, 2, 16) STAP_BS(3, 3, 16) STAP_BS(5, 2, 16) STAP_BS(5, 3, 16)
#undef STAP_BS
  return hipErrorInvalidValue;
}

}  // namespace stap
