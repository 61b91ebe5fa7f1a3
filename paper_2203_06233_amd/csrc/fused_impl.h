// Fused covariance -> Cholesky -> solve per system (the path of stap_run):
// the loaded covariance of a (Doppler bin, training block) never leaves the
// compute unit.
//   phase 1  cov_accumulate() (cov_impl.h) on MFMA; the FP64 trace gives
//            delta;
//   phase 2  the blocked solve, bsolve_blocks() (bsolve_impl.h), starts on the
//            accumulators (bfused_system() below), or the column sweep,
//            solve_system() (solve_impl.h), reads the packed lower triangle of
//            R_L that phase 1 left in LDS over the snapshot staging buffer.
// With refinement R_L stays in LDS for the FP64 residual, as blocks or packed.
// Compared with the stage kernels this saves the covariance round trip
// through HBM (P*B*D*D*8 bytes written and half of it read back).
#pragma once

#include "bsolve_impl.h"
#include "common.h"
#include "cov_impl.h"
#include "kernels.h"
#include "solve_impl.h"

namespace stap {


struct PackedR {
  const float2* Rp;
  __device__ float2 lower(int i, int k) const { return Rp[i * (i + 1) / 2 + k]; }
};

// System `sys` of one cube: wout and info_out are the cube's arrays.
template <int TY, int NA, int NB, int NVS, int MODE, bool REFINE>
__device__ __forceinline__ void fused_system(const float2* __restrict__ snap, const float2* __restrict__ steer,
                                             float2* __restrict__ wout, int* __restrict__ info_out,
                                             const Dims& d, int sys) {
  using K = SolveCfg<TY, NA, NB, NVS>;
  using C = CovCfg<K::DPC, K::NT / 64, MODE>;
  constexpr int PACK = (K::kPacked + (REFINE ? K::kSlab : 0)) * 8;  // packed R_L (+ residual slab)
  constexpr int BYTES = C::LDS_BYTES > PACK ? C::LDS_BYTES : PACK;
  __shared__ __align__(16) unsigned char lds[BYTES];
  __shared__ SolveShared<K> sh;
  __shared__ double dsum[K::DPC];
  __shared__ float red[K::NT / 64];

  const int k = sys / d.B, b = sys - (sys / d.B) * d.B;
  const int D = d.D;
  const float2* X = snap + (long long)k * D * d.R;
  floatx4 accR[C::TPW], accI[C::TPW];
  int tI[C::TPW], tJ[C::TPW];
  cov_tiles<C>(tI, tJ);
  cov_accumulate<C>(X, d.R, D, d.N, train_cells(d, b), lds, red, tI, tJ, accR, accI);
  const float dl = cov_delta<C>(accR, tI, tJ, D, d.eps, dsum);
  __syncthreads();  // the staging buffer is dead: reuse it for R_L
  float2* Rp = reinterpret_cast<float2*>(lds);
  cov_emit<C>(accR, accI, tI, tJ, D, dl, [&](int row, int col, float2 v) { Rp[row * (row + 1) / 2 + col] = v; });
  __syncthreads();
  solve_system<K, REFINE, true>(PackedR{Rp}, Rp, Rp + K::kPacked, steer + steer_offset(d, sys),
                                wout + (long long)sys * d.S * D,
                                info_out ? info_out + sys : nullptr, d, sh);
}


// Register budgets (waves per SIMD) of the one-cube column sweep without
// refinement that are met without spills and that the compiler's own choice
// misses: one block column with split-BF16 covariance (12 DOF, 30 vectors, 4096
// systems: 58.7 us with 90 registers, 52.7 with 80) and three with more than
// 32 steering vectors on FP32 (48 DOF, 64 vectors: 346 us with 98, 316 with 96).
template <int TY, int NB, int NVS, int MODE, bool REFINE>
constexpr int fused_min_waves() {
  if (TY != 16 || REFINE) return 1;
  return NB == 1 && MODE == 1 ? 6 : NB == 3 && NVS == 4 && MODE == 0 ? 5 : 1;
}

template <int TY, int NA, int NB, int NVS, int MODE, bool REFINE>
__global__ __launch_bounds__(16 * TY) __attribute__((amdgpu_waves_per_eu(fused_min_waves<TY, NB, NVS, MODE, REFINE>())))
void fused_kernel(const float2* __restrict__ snap,
                                                        const float2* __restrict__ steer,
                                                        float2* __restrict__ wout, int* __restrict__ info_out,
                                                        Dims d) {
  fused_system<TY, NA, NB, NVS, MODE, REFINE>(snap, steer, wout, info_out, d, blockIdx.x);
}

// Persistent workgroups take the next system from a device work queue: one
// 64-bit counter (reset by the launch that writes the problem table) that
// each workgroup advances atomically when it finishes a system.  Cubes are
// ordered by cost (largest first), so the most expensive systems are handed
// out first and the cheap ones fill in behind them.  Every workgroup leaves
// when the counter has passed the last system.
__device__ __forceinline__ long long next_system(unsigned long long* queue, long long* slot) {
  if (lane_tid() == 0) *slot = (long long)atomicAdd(queue, 1ULL);
  __syncthreads();
  const long long g = *slot;
  __syncthreads();  // every thread has read the slot before the next claim overwrites it
  return g;
}

template <int TY, int NA, int NB, int NVS, int MODE, bool REFINE>
__global__ __launch_bounds__(16 * TY) void fused_batched_kernel(const ProbDesc* __restrict__ desc, int n,
                                                                long long total, unsigned long long* queue) {
  __shared__ long long slot;
  for (long long g = next_system(queue, &slot); g < total; g = next_system(queue, &slot)) {
    int lo = 0, hi = n - 1;
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (desc[mid].sys_begin <= g) lo = mid;
      else hi = mid - 1;
    }
    const ProbDesc& pd = desc[lo];
    const Dims d = pd.d;
    fused_system<TY, NA, NB, NVS, MODE, REFINE>(pd.snap, pd.steer, pd.w, pd.info, d, (int)(g - pd.sys_begin));
    __syncthreads();
  }
}

// R_L in LDS for the residual of the blocked solve: the blocks of the lower
// block triangle in their register order, both triangles of a diagonal block.
struct LdsR {
  const float* base;
  int NB;
  __device__ __forceinline__ Acc get(int J, int I, int nat) const {
    if (J <= I) {  // R[16J + 4q + s][16I + m] = conj(R[16I + m][16J + 4q + s])
      Acc a = blk_load(base + lblock(NB, I, J) * kBlk, nat);
      a.im = -a.im;
      return a;
    }
    return blk_load_t(base + lblock(NB, J, I) * kBlk);
  }
};

// The same with the blocked matrix-core solve (bsolve_impl.h): NB block
// columns of the covariance (compile time, for the covariance tiles), NS
// steering blocks at most, NW waves, NSL / NSM register blocks per wave.  A
// wave computes the covariance tiles of the very blocks it owns in the solve,
// in the solve's register order (operands swapped), so the factorisation
// starts on the accumulators: going through a packed copy in LDS instead took
// 14 % of the kernel (39 of 274 thousand cycles per system at 96 DOF).  With
// refinement the blocks are also stored in LDS for the FP64 residual and the
// solver's exchange blocks follow them; without, those reuse the staging
// bytes.
template <int NB, int NS, int NSL, int NSM, int NW, int MODE, int LEVEL>
__device__ __forceinline__ void bfused_system(const float2* __restrict__ snap, const float2* __restrict__ steer,
                                              float2* __restrict__ wout, int* __restrict__ info_out,
                                              const Dims& d, int sys) {
  constexpr bool REFINE = LEVEL != kPlain;
  using C = CovCfg<16 * NB, NW, MODE>;
  using B = BCfg<NSL, NSM, NW>;
  static_assert(C::TPW == NSL, "one covariance tile per L slot");
  constexpr int RBYTES = NB * (NB + 1) / 2 * kBlk * 4;
  constexpr int EXCH = (int)B::lds_bytes(NB, NS, LEVEL);
  constexpr int B2 = REFINE ? RBYTES + EXCH : EXCH;
  constexpr int BYTES = C::LDS_BYTES > B2 ? C::LDS_BYTES : B2;
  __shared__ __align__(16) unsigned char lds[BYTES];
  __shared__ double dsum[16 * NB];
  __shared__ float red[NW];

  const int k = sys / d.B, b = sys - (sys / d.B) * d.B;
  const int D = d.D;
  const float2* X = snap + (long long)k * D * d.R;
  const float2* V = steer + steer_offset(d, sys);
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const Slots<B> sl(D, d.S, wave);
  floatx4 accR[NSL], accI[NSL];
  int tI[NSL], tJ[NSL];
#pragma unroll
  for (int t = 0; t < NSL; ++t) {
    tI[t] = sl.lv[t] ? sl.lr[t] : -1;
    tJ[t] = sl.lc[t];
  }
  cov_accumulate<C, true>(X, d.R, D, d.N, train_cells(d, b), lds, red, tI, tJ, accR, accI);
  Acc al[NSL], am[NSM];
  load_steer(sl, V, D, d.S, am);  // in flight across the trace
  float mean;
  const float dl = cov_delta<C>(accR, tI, tJ, D, d.eps, dsum, &mean);  // its barrier retires the staging buffer
  const SysScale sc(REFINE ? mean + dl : 1.f);

  float* const Rb = reinterpret_cast<float*>(lds);
  const SolveLds<B, LEVEL> L(lds + (REFINE ? RBYTES : 0), sl.NB, sl.NS);
  const int lane = lane_tid() & 63, m = lane & 15, q = lane >> 4, nat = nat_ofs();
#pragma unroll
  for (int t = 0; t < NSL; ++t) {
    al[t].re = accR[t];
    al[t].im = accI[t];
    if (sl.lv[t]) {
      float* const blk = REFINE ? Rb + lblock(sl.NB, sl.lr[t], sl.lc[t]) * kBlk : L.xb + sl.lr[t] * kBlk;
      if (sl.lr[t] == sl.lc[t]) {
        // both triangles from the lower one, diagonal real with the loading,
        // identity beyond D; a wave's LDS accesses keep their order
        blk_store(blk, al[t], nat);
        const Acc T = blk_load_t(blk);
        const int r = 16 * sl.lr[t] + m;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int c = 4 * q + i;
          if (c > m) {
            al[t].re[i] = T.re[i];
            al[t].im[i] = -T.im[i];
          } else if (c == m) {
            al[t].re[i] = r < D ? al[t].re[i] + dl : 1.f;
            al[t].im[i] = 0.f;
            L.rdiag[r] = al[t].re[i];
          }
        }
      }
      if (REFINE) {
        blk_store(blk, al[t], nat);
        // (the identity beyond D scales with the rest)
        al[t] = acc_scale(al[t], -sc.r);
      } else {
        al[t] = acc_neg(al[t]);
      }
    }
  }
  for (int r = threadIdx.x; r < 16 * sl.NB; r += B::NT) L.d64[r] = 0.0;
  // the R_L blocks are dead after the last residual: u of that step is kept
  // there when it fits (their number at run time covers NS NB blocks)
  const bool park = REFINE && sl.NB + 1 >= 2 * sl.NS;
  bsolve_blocks<B, LEVEL>(sl, al, am, L, LdsR{Rb, sl.NB}, V, wout + (long long)sys * d.S * D,
                           info_out ? info_out + sys : nullptr, d, park ? Rb : nullptr, sc);
}

// Register budgets (waves per SIMD) that the kernels meet with no or few
// spills: 128 registers with 8 waves and up to 6 block columns, so that two
// systems share a compute unit (7 registers spill; with 4 steering blocks 146
// are taken, and the 97 KB of LDS leave room for one system anyway), with 4
// waves up to 3 and with one wave; 168 with 4 waves and 4 block columns and
// with 2 waves.
template <int NB, int NS, int NW>
constexpr int bfused_min_waves() {
  if (NW == 8 && NB <= 6) return 4;
  if (NW == 4 && NS <= 2) return NB <= 3 ? 4 : NB == 4 ? 3 : 1;
  if (NW == 1 && NS <= 2) return 4;
  return NW <= 2 ? 3 : 1;
}

template <int NB, int NS, int NSL, int NSM, int NW, int MODE, int LEVEL>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(bfused_min_waves<NB, NS, NW>())))
void bfused_kernel(const float2* __restrict__ snap,
                                                         const float2* __restrict__ steer,
                                                         float2* __restrict__ wout, int* __restrict__ info_out,
                                                         Dims d) {
  bfused_system<NB, NS, NSL, NSM, NW, MODE, LEVEL>(snap, steer, wout, info_out, d, blockIdx.x);
}

template <int NB, int NS, int NSL, int NSM, int NW, int MODE, int LEVEL>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(bfused_min_waves<NB, NS, NW>())))
void bfused_batched_kernel(const ProbDesc* __restrict__ desc, int n,
                                                                 long long total, unsigned long long* queue) {
  __shared__ long long slot;
  for (long long g = next_system(queue, &slot); g < total; g = next_system(queue, &slot)) {
    int lo = 0, hi = n - 1;
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (desc[mid].sys_begin <= g) lo = mid;
      else hi = mid - 1;
    }
    const ProbDesc& pd = desc[lo];
    const Dims d = pd.d;
    bfused_system<NB, NS, NSL, NSM, NW, MODE, LEVEL>(pd.snap, pd.steer, pd.w, pd.info, d, (int)(g - pd.sys_begin));
    __syncthreads();
  }
}

template <int TY, int NA, int NB, int NVS, int MODE>
hipError_t go_fused_batched(const ProbDesc* desc, int n, long long total, int refine, hipStream_t st,
                            unsigned long long* queue) {
  // enough workgroups to fill every CU a few times over, never more than systems
  const long long want = 256LL * (TY == 16 ? 4 : 2);
  const dim3 grid((unsigned)(total < want ? total : want)), block(16 * TY);
  if (refine == 0)
    hipLaunchKernelGGL((fused_batched_kernel<TY, NA, NB, NVS, MODE, false>), grid, block, 0, st, desc, n, total,
                       queue);
  else
    hipLaunchKernelGGL((fused_batched_kernel<TY, NA, NB, NVS, MODE, true>), grid, block, 0, st, desc, n, total,
                       queue);
  return hipGetLastError();
}

template <int TY, int NA, int NB, int NVS, int MODE>
hipError_t go_fused(const Dims& d, const float2* snap, const float2* steer, float2* w, int* info,
                    hipStream_t st) {
  const dim3 grid(d.P * d.B), block(16 * TY);
  if (d.refine == 0)
    hipLaunchKernelGGL((fused_kernel<TY, NA, NB, NVS, MODE, false>), grid, block, 0, st, snap, steer, w, info, d);
  else
    hipLaunchKernelGGL((fused_kernel<TY, NA, NB, NVS, MODE, true>), grid, block, 0, st, snap, steer, w, info, d);
  return hipGetLastError();
}

}  // namespace stap
