// Blocked Cholesky solve of one system inside one wave, every block held in
// that wave's registers for the whole solve (up to NB = 6 block columns of
// R_L and NS = 2 blocks of steering vectors: D <= 96, S <= 32), without
// refinement.
//
// The steps and the block algebra are those of bsolve_blocks()
// (bsolve_impl.h): right-looking factorisation with the in-wave diagonal
// factor-and-invert, the forward solve of the steering rows M = V^H riding
// along as extra rows, and the back solve in row form Z L = Y^H.  What
// differs is the placement: with the block coordinates known at compile time every loop is
// unrolled, the operands of a block product are read straight from the
// registers of the blocks they come from (no exchange through LDS and no
// barrier), and the only LDS traffic is the transposition of the L blocks a
// back-solve step multiplies by.
// One wave per system leaves the four SIMDs of a compute unit on four
// systems at once; the instruction stream of the wave interleaves the
// serial diagonal work with the matrix-core products of the same step.
#pragma once

#include "bsolve_impl.h"

namespace stap {
namespace wsv {

constexpr int tri(int I, int J) { return I * (I + 1) / 2 + J; }

// Back solve in row form, Z L = Y^H (M holds Y^H on entry, Z on exit): for J
// descending, Z_J = M_J Linv_JJ, then M_I -= Z_J L_JI for I < J.  The
// transposes of row J of L pass through LDS (tb, SLOTS blocks), SLOTS at a
// time, the diagonal block first.
template <int NB, int NS, int SLOTS>
__device__ __forceinline__ void back_solve(const Acc (&L)[NB * (NB + 1) / 2], Acc (&M)[NS * NB], float* tb, int nat) {
#pragma unroll
  for (int J = NB - 1; J >= 0; --J) {
#pragma unroll
    for (int I0 = J; I0 >= 0; I0 -= SLOTS) {
      __syncthreads();  // earlier reads of tb are done
#pragma unroll
      for (int g = 0; g < SLOTS && I0 - g >= 0; ++g) blk_store_t(tb + g * kBlk, L[tri(J, I0 - g)]);
      __syncthreads();
#pragma unroll
      for (int g = 0; g < SLOTS && I0 - g >= 0; ++g) {
        const int I = I0 - g;
        const Acc Lt = blk_load(tb + g * kBlk, nat);
        if (I == J) {
#pragma unroll
          for (int N = 0; N < NS; ++N) {
            Acc x = acc_zero();
            mma_pq<false>(x, M[N * NB + J], Lt);
            M[N * NB + J] = x;
          }
        } else {
#pragma unroll
          for (int N = 0; N < NS; ++N) mma_pq<true>(M[N * NB + I], M[N * NB + J], Lt);
        }
      }
    }
  }
}

// Forward solve Y^H L^H = M with the factor in L (Linv_JJ on the diagonal):
// M_J := M_J Linv_JJ^H, then M_K -= M_J L_KJ^H for K > J, block by block in
// the order of the factorisation's own updates of M.
template <int NB, int NS>
__device__ __forceinline__ void forward_solve(const Acc (&L)[NB * (NB + 1) / 2], Acc (&M)[NS * NB]) {
#pragma unroll
  for (int J = 0; J < NB; ++J) {
#pragma unroll
    for (int N = 0; N < NS; ++N) {
      Acc x = acc_zero();
      mma_pqh<false>(x, M[N * NB + J], L[tri(J, J)]);
      M[N * NB + J] = x;
    }
#pragma unroll
    for (int K = J + 1; K < NB; ++K)
#pragma unroll
      for (int N = 0; N < NS; ++N) mma_pqh<true>(M[N * NB + K], M[N * NB + J], L[tri(K, J)]);
  }
}

// The trailing updates of factorisation step J other than the one of
// diagonal block J+1, numbered 0..COUNT-1: first the L blocks (I, K),
// K = J+1.., I = K.., then the M blocks (N, K).
template <int NB, int NS, int J>
struct StepWork {
  static constexpr int NLU = (NB - J - 1) * (NB - J) / 2 - (J + 1 < NB ? 1 : 0);
  static constexpr int COUNT = NLU + (NB - J - 1) * NS;
  struct Item {
    bool isL;
    int I, K, N;
  };
  static constexpr Item item(int p) {
    int n = 0;
    for (int K = J + 1; K < NB; ++K)
      for (int I = K; I < NB; ++I) {
        if (K == J + 1 && I == J + 1) continue;
        if (n == p) return Item{true, I, K, 0};
        ++n;
      }
    for (int K = J + 1; K < NB; ++K)
      for (int N = 0; N < NS; ++N) {
        if (n == p) return Item{false, 0, K, N};
        ++n;
      }
    return Item{false, -1, -1, -1};
  }
};

template <int NB, int NS, int J, int P, int END>
__device__ __forceinline__ void step_work(Acc (&L)[NB * (NB + 1) / 2], Acc (&M)[NS * NB]) {
  if constexpr (P < END) {
    constexpr auto it = StepWork<NB, NS, J>::item(P);
    if constexpr (it.isL) mma_pqh<true>(L[tri(it.I, it.K)], L[tri(it.I, J)], L[tri(it.K, J)]);
    else mma_pqh<true>(M[it.N * NB + it.K], M[it.N * NB + J], L[tri(it.K, J)]);
    step_work<NB, NS, J, P + 1, END>(L, M);
  }
}

// Columns j.. of diag_factor_inv() with the share of step J's trailing
// updates that goes with each column issued right after it, so the wave's
// instruction stream interleaves the serial VALU work of diagonal block
// J+1 with independent matrix-core products.
template <int NB, int NS, int J, int j>
__device__ __forceinline__ void diag_cols_work(Diag<false>& s, Acc (&L)[NB * (NB + 1) / 2], Acc (&M)[NS * NB]) {
  constexpr int C = StepWork<NB, NS, J>::COUNT;
  diag_col<j>(s);
  step_work<NB, NS, J, j * C / 16, (j + 1) * C / 16>(L, M);
  if constexpr (j < 15) diag_cols_work<NB, NS, J, j + 1>(s, L, M);
}

// Factorisation step J (diagonal block J already holds Linv_JJ): panel,
// the update and factorisation of diagonal block J+1 interleaved with the
// remaining updates of the step, then step J+1.  d64 (LDS) collects the
// FP64 row sums of |L|^2 over the finished block columns and rdiag holds
// the loaded diagonal: the FP64 pivots of block J+1 start from their
// difference.
template <int NB, int NS, int J>
__device__ __forceinline__ void fact_step(Acc (&L)[NB * (NB + 1) / 2], Acc (&M)[NS * NB], int& fail, double* d64,
                                          const float* rdiag) {
  const int lane = lane_tid() & 63;
#pragma unroll
  for (int I = J + 1; I < NB; ++I) {
    Acc x = acc_zero();
    mma_pqh<false>(x, L[tri(I, J)], L[tri(J, J)]);
    L[tri(I, J)] = x;
    const double pn = blk_row_norm2(x);
    if (lane < 16) d64[16 * I + lane] += pn;
  }
#pragma unroll
  for (int N = 0; N < NS; ++N) {
    Acc x = acc_zero();
    mma_pqh<false>(x, M[N * NB + J], L[tri(J, J)]);
    M[N * NB + J] = x;
  }
  if constexpr (J + 1 < NB) {
    mma_pqh<true>(L[tri(J + 1, J + 1)], L[tri(J + 1, J)], L[tri(J + 1, J)]);
    const int m = lane & 15;
    Diag<false> s;
    diag_begin(s, L[tri(J + 1, J + 1)], (double)rdiag[16 * (J + 1) + m] - d64[16 * (J + 1) + m]);
    diag_cols_work<NB, NS, J, 0>(s, L, M);
    fail = (fail == 0 && s.fail != 0) ? 16 * (J + 1) + s.fail : fail;
    L[tri(J + 1, J + 1)] = diag_end<1>(s);
    fact_step<NB, NS, J + 1>(L, M, fail, d64, rdiag);
  }
}

// LDS of one system: transpose slots, then the FP64 row sums of |L|^2 (16 NB
// doubles) and the loaded diagonal (16 NB floats) for the pivots.
template <int NB>
struct WsLds {
  static constexpr int SLOTS = NB;
  static constexpr int PIV = 16 * NB + 8 * NB;  // in complex (8-byte) units
  static constexpr int COMPLEX = SLOTS * kBlk / 2 + PIV;
};

// Elements k .. k+3 of row s of a [rows][D] array, zero outside it; TAIL if
// columns from D on can be among them.  The loads are at clamped indices and
// behind no branch, so those of all blocks are in flight together (a bounds
// check around each costs a memory latency per block: the 16 x 128 x 4096
// cube, 48 DOF, 274 us per pass with those, 262 without; 96 DOF, 32768
// systems, 5.24 and 5.06-5.20 ms).
template <bool TAIL>
__device__ __forceinline__ void load_row4(const float2* __restrict__ base, int s, int k, int rows, int D, float2 (&v)[4]) {
  typedef float f4 __attribute__((ext_vector_type(4), aligned(8)));
  const bool row_ok = s < rows;
  const float2* const p = base + min(s, rows - 1) * D;
  if (TAIL) {
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = p[min(k + i, D - 1)];
  } else {
    const f4 a = *reinterpret_cast<const f4*>(p + k), b = *reinterpret_cast<const f4*>(p + k + 2);
    v[0] = make_float2(a.x, a.y);
    v[1] = make_float2(a.z, a.w);
    v[2] = make_float2(b.x, b.y);
    v[3] = make_float2(b.z, b.w);
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const bool ok = row_ok & (!TAIL | (k + i < D));
    v[i].x = ok ? v[i].x : 0.f;
    v[i].y = ok ? v[i].y : 0.f;
  }
}

// M = V^H of steering rows 16 N0 .. on.
template <int NB, int NS>
__device__ __forceinline__ void load_m(const float2* __restrict__ steer, int N0, int D, int S, Acc (&M)[NS * NB]) {
  const int lane = lane_tid() & 63, m = lane & 15, q = lane >> 4;
#pragma unroll
  for (int N = 0; N < NS; ++N) {
#pragma unroll
    for (int J = 0; J < NB; ++J) {
      const int s = 16 * (N0 + N) + m;
      float2 v[4];
      if (J == NB - 1) load_row4<true>(steer, s, 16 * J + 4 * q, S, D, v);
      else load_row4<false>(steer, s, 16 * J + 4 * q, S, D, v);
      Acc a;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        a.re[i] = v[i].x;
        a.im[i] = -v[i].y;
      }
      M[N * NB + J] = a;
    }
  }
}

// From Y^H in M to the weights of steering rows 16 N0 .. on: gamma_s =
// ||y_s||^2 summed over the row's blocks, back solve, w_s = u_s /
// sqrt(gamma_s) with u_s = conj(z_s).
template <int NB, int NS>
__device__ __forceinline__ void finish_m(const Acc (&L)[NB * (NB + 1) / 2], Acc (&M)[NS * NB], int N0,
                                         float2* __restrict__ W, int D, int S, float* tb, int nat) {
  const int lane = lane_tid() & 63, m = lane & 15, q = lane >> 4;
  double gam[NS];
#pragma unroll
  for (int N = 0; N < NS; ++N) {
    gam[N] = 0.0;
#pragma unroll
    for (int J = 0; J < NB; ++J) {
      const Acc& y = M[N * NB + J];
      float p = 0.f;
#pragma unroll
      for (int i = 0; i < 4; ++i) p = fmaf(y.re[i], y.re[i], fmaf(y.im[i], y.im[i], p));
      p += __shfl_xor(p, 16);
      p += __shfl_xor(p, 32);
      gam[N] += p;
    }
  }
  back_solve<NB, NS, WsLds<NB>::SLOTS>(L, M, tb, nat);
  const bool vec = rows16(W, D);
#pragma unroll
  for (int N = 0; N < NS; ++N) {
    const int s = 16 * (N0 + N) + m;
    const float sc = 1.f / sqrtf((float)gam[N]);
#pragma unroll
    for (int J = 0; J < NB; ++J) {
      float2 w[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) w[i] = make_float2(M[N * NB + J].re[i] * sc, -M[N * NB + J].im[i] * sc);
      store4(W, s, 16 * J + 4 * q, s < S, D, vec, w);
    }
  }
}

// Steering blocks in registers at a time: with 6 block columns two of them
// (264 registers with L) leave one wave on a SIMD, which waits out every
// dependency; one fits two waves.
constexpr int steer_group(int NB, int NS) { return NB >= 5 ? 1 : NS; }

// Solve one system: R is its loaded covariance, of which the lower triangle is
// read, [D][D] row-major, W its [S][D] weights, info its status word (may be null);
// D <= 16 NB, S <= 16 NS.  lds points at WsLds<NB>::COMPLEX complex of
// 16-byte aligned LDS.  Blocks beyond D carry the identity, steering rows
// beyond S are zero.  The first group of steering blocks rides along with the
// factorisation, the others take their forward solve from the stored factor.
template <int NB, int NS>
__device__ __forceinline__ void wsolve_system(const float2* __restrict__ R, const float2* __restrict__ steer,
                                              float2* __restrict__ W, int* __restrict__ info, const Dims& d,
                                              float2* lds) {
  constexpr int NL = NB * (NB + 1) / 2, G = steer_group(NB, NS);
  const int D = d.D, S = d.S;
  const int lane = lane_tid() & 63, m = lane & 15, q = lane >> 4;
  float* tb = reinterpret_cast<float*>(lds);
  const int nat = nat_ofs();
  double* d64 = reinterpret_cast<double*>(tb + WsLds<NB>::SLOTS * kBlk);
  float* rdiag = reinterpret_cast<float*>(d64 + 16 * NB);
  for (int r = lane; r < 16 * NB; r += 64) d64[r] = 0.0;

  Acc L[NL], M[G * NB];
#pragma unroll
  for (int I = 0; I < NB; ++I) {
#pragma unroll
    for (int J = 0; J <= I; ++J) {
      const int r = 16 * I + m;
      Acc a;
      float2 v[4];
      if (J == NB - 1) load_row4<true>(R, r, 16 * J + 4 * q, D, D, v);
      else load_row4<false>(R, r, 16 * J + 4 * q, D, D, v);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int c = 16 * J + 4 * q + i;
        a.re[i] = I == J && r >= D && c == r ? 1.f : v[i].x;
        a.im[i] = v[i].y;
        if (I == J && c == r) rdiag[r] = a.re[i];
      }
      L[tri(I, J)] = a;
    }
  }
  load_m<NB, G>(steer, 0, D, S, M);
  // both triangles of the diagonal blocks from the lower one, diagonal real; a
  // wave's LDS accesses keep their order (reading the mirrored elements from
  // memory instead costs 5 % of the solve)
#pragma unroll
  for (int I = 0; I < NB; ++I) {
    float* const blk = tb + I * kBlk;
    Acc a = L[tri(I, I)];
    blk_store(blk, a, nat);
    const Acc T = blk_load_t(blk);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int c = 4 * q + i;
      a.re[i] = c > m ? T.re[i] : a.re[i];
      a.im[i] = c > m ? -T.im[i] : c == m ? 0.f : a.im[i];
    }
    L[tri(I, I)] = a;
  }

  // ---- factorisation with the forward solve of the first steering rows
  int fail = 0;
  {
    Acc X;
    float unused;
    fail = diag_factor_inv<1, false>(L[0], X, unused, (double)blk_diag(L[0]), nullptr, nullptr);
    L[0] = X;
  }
  fact_step<NB, G, 0>(L, M, fail, d64, rdiag);
  if (fail) {
    for (int e = lane; e < S * D; e += 64) W[e] = make_float2(0.f, 0.f);
    if (lane == 0 && info) *info = fail;
    return;
  }
  finish_m<NB, G>(L, M, 0, W, D, S, tb, nat);
#pragma unroll 1
  for (int N0 = G; 16 * N0 < S; N0 += G) {
    load_m<NB, G>(steer, N0, D, S, M);
    forward_solve<NB, G>(L, M);
    finish_m<NB, G>(L, M, N0, W, D, S, tb, nat);
  }
  if (lane == 0 && info) *info = 0;
}

}  // namespace wsv
}  // namespace stap
