// Blocked Cholesky solve of one system on the matrix cores.
//
// The loaded covariance R_L (D x D, padded to 16 NB with an identity tail)
// and the conjugated steering rows M = V^H (S x D, padded to 16 NS rows with
// zeros) are cut into 16 x 16 complex blocks.  Each block lives in the
// registers of one wave for the whole solve (static round-robin ownership),
// so the right-looking updates never move the block they update; only the
// operands of a step pass through LDS.
//
//   factorisation  for each block column J: the owner of the diagonal block
//                  factors it (16 sequential columns inside one wave) and
//                  forms its triangular inverse Linv_JJ; the owners of the
//                  panel blocks form L_IJ = A_IJ Linv_JJ^H (and M_NJ :=
//                  M_NJ Linv_JJ^H, the forward solve riding along as extra
//                  rows); every later block X takes X -= P Q^H with P, Q
//                  from the published panel.  M ends as Y^H = (L^-1 V)^H.
//   gamma          gamma_s = ||y_s||^2.
//   back solve     in row form Z L = Y^H with Z = U^H: for J descending,
//                  Z_J = M_J Linv_JJ, then M_I -= Z_J L_JI for I < J.
//   output         w_s = u_s / sqrt(gamma_s), u_s = conj(row s of Z).
//
// Block products are 16 x 16 x 16 complex: without refinement four real
// 16 x 16 x 4 FP32 MFMAs per k-quarter (OpF32), with refinement six
// 16 x 16 x 32 BF16 MFMAs per component (OpSplit).  Fragment layout (lane l, m = l % 16, q = l / 16): the lane holds
// X[m][4q + i], i = 0..3.  This is the MFMA result layout of X^T, and the A
// and B operand layouts of a product whose k index runs over the block
// columns, so every product is formed transposed (X^T -= conj(Q) P^T) and no
// block is ever shuffled.
//
// In LDS a block is two planes of 256 floats (real, imaginary), so a fragment
// moves as two 16-byte accesses per lane straight from and to the registers
// of the products.  Within a plane the 16-byte unit of row r, columns
// 4c .. 4c+3 sits at 16 c + 4 (r / 4) + (r + c) % 4: the 16 lanes of a
// fragment access and the 64 lanes of a transposed one (bofs) both fall on
// distinct banks.  The interleaved complex layout before it needed register
// moves around every access, and its transposed accesses fell eight lanes to
// a bank.
#pragma once

#include <type_traits>

#include "common.h"

namespace stap {

struct Acc {
  floatx4 re, im;
};

constexpr int kBlk = 512;  // floats of one block in LDS

// Offset of element (r, c) in a plane of a block.
__device__ __forceinline__ int bofs(int r, int c) {
  const int cq = c >> 2;
  return 4 * (16 * cq + 4 * (r >> 2) + ((r + cq) & 3)) + (c & 3);
}
// Offset of the lane's own X[m][4q .. 4q+3].
__device__ __forceinline__ int nat_ofs() {
  const int l = lane_tid() & 63;
  return bofs(l & 15, 4 * (l >> 4));
}

__device__ __forceinline__ Acc blk_load(const float* blk, int nat) {
  Acc a;
  a.re = *reinterpret_cast<const floatx4*>(blk + nat);
  a.im = *reinterpret_cast<const floatx4*>(blk + 256 + nat);
  return a;
}
__device__ __forceinline__ void blk_store(float* blk, const Acc& a, int nat) {
  *reinterpret_cast<floatx4*>(blk + nat) = a.re;
  *reinterpret_cast<floatx4*>(blk + 256 + nat) = a.im;
}
// Store X^T: the lane's X[m][4q + i] goes to element (4q + i, m).
__device__ __forceinline__ void blk_store_t(float* blk, const Acc& a) {
  const int l = lane_tid() & 63, m = l & 15, q = l >> 4;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int o = bofs(4 * q + i, m);
    blk[o] = a.re[i];
    blk[256 + o] = a.im[i];
  }
}
// The lane's X[4q + i][m], i = 0..3.
__device__ __forceinline__ Acc blk_load_t(const float* blk) {
  const int l = lane_tid() & 63, m = l & 15, q = l >> 4;
  Acc a;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int o = bofs(4 * q + i, m);
    a.re[i] = blk[o];
    a.im[i] = blk[256 + o];
  }
  return a;
}
__device__ __forceinline__ Acc acc_zero() {
  Acc a;
  a.re = floatx4{0.f, 0.f, 0.f, 0.f};
  a.im = floatx4{0.f, 0.f, 0.f, 0.f};
  return a;
}

__device__ __forceinline__ floatx4 mfma4(float a, float b, floatx4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// x -= P Q^H (SUB) or x += P Q^H.  As x^T -/+= conj(Q) P^T: MFMA A operand
// conj(Q)[m][k], B operand P[m][k], k-quarter s covering k = 4 q' + s.
template <bool SUB>
__device__ __forceinline__ void mma_pqh(Acc& x, const Acc& P, const Acc& Q) {
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    const float qr = SUB ? -Q.re[s] : Q.re[s], qi = SUB ? -Q.im[s] : Q.im[s];
    x.re = mfma4(qr, P.re[s], x.re);  // Re(conj(q) p) = qr pr + qi pi
    x.re = mfma4(qi, P.im[s], x.re);
    x.im = mfma4(qr, P.im[s], x.im);  // Im(conj(q) p) = qr pi - qi pr
    x.im = mfma4(-qi, P.re[s], x.im);
  }
}

// x -= P Q (SUB) or x += P Q, with Qt the fragment of Q^T.  As x^T -/+= Q^T P^T.
template <bool SUB>
__device__ __forceinline__ void mma_pq(Acc& x, const Acc& P, const Acc& Qt) {
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    const float qr = SUB ? -Qt.re[s] : Qt.re[s], qi = SUB ? -Qt.im[s] : Qt.im[s];
    x.re = mfma4(qr, P.re[s], x.re);  // Re(q p) = qr pr - qi pi
    x.re = mfma4(-qi, P.im[s], x.re);
    x.im = mfma4(qr, P.im[s], x.im);  // Im(q p) = qr pi + qi pr
    x.im = mfma4(qi, P.re[s], x.im);
  }
}

// How the blocked solve forms its block products x += P Q^H and x += P Q.
//
// Without refinement: FP32 MFMA on the blocks themselves.
//
// With refinement: every published block is split exactly into three BF16
// terms per component (x = h + m + l to 24 bits, as in the covariance) and
// the six products hh, hm, mh, hl, lh, mm run on v_mfma_f32_16x16x32_bf16
// with FP32 accumulation; a lane's eight values (four real, four imaginary)
// are its k slice of one 32-deep product, so a complex block product is 12
// instructions of 16 cycles instead of 16 of 32.  What decides is the unit,
// not the cycles: FP32 (and FP64) MFMA occupies the vector ALU of its SIMD,
// and while one wave streams it no other wave of the SIMD issues a VALU
// instruction at any priority (measured: a wave's FMA goes from 5 cycles to
// waiting until the stream ends; beside BF16 MFMA it takes 8), so the waves'
// products froze the diagonal factorisation that everything else waits for.
// The split form is the more exact of the two: against 64 bits, one refinement
// step, on the same factorisation, 60 DOF 1.9e-6 with FP32 products and 1.5e-6
// split, 96 DOF 1.2e-6 and 0.8e-6, 192 DOF 8.8e-7 and 5.2e-7.  Without
// refinement the FP32 products stay as they are.
struct OpF32 {
  typedef Acc Frag;
  static constexpr int kB = kBlk;  // floats of a published block
  static __device__ __forceinline__ Frag frag(const Acc& a) { return a; }
  static __device__ __forceinline__ Frag load(const float* blk, int nat) { return blk_load(blk, nat); }
  static __device__ __forceinline__ void store(float* blk, const Frag& f, int nat) { blk_store(blk, f, nat); }
  static __device__ __forceinline__ void pqh(Acc& x, const Frag& P, const Frag& Q) { mma_pqh<false>(x, P, Q); }
  static __device__ __forceinline__ void pq(Acc& x, const Frag& P, const Frag& Qt) { mma_pq<false>(x, P, Qt); }
};
struct OpSplit {
  struct Frag {
    uint4 t[3];  // terms h, m, l: {re 0-1, re 2-3, im 0-1, im 2-3}
  };
  static constexpr int kB = 768;  // three planes of 64 16-byte units
  static __device__ __forceinline__ Frag frag(const Acc& a) {
    Frag f;
    split3x2(a.re[0], a.re[1], f.t[0].x, f.t[1].x, f.t[2].x);
    split3x2(a.re[2], a.re[3], f.t[0].y, f.t[1].y, f.t[2].y);
    split3x2(a.im[0], a.im[1], f.t[0].z, f.t[1].z, f.t[2].z);
    split3x2(a.im[2], a.im[3], f.t[0].w, f.t[1].w, f.t[2].w);
    return f;
  }
  static __device__ __forceinline__ Frag load(const float* blk, int nat) {
    Frag f;
#pragma unroll
    for (int p = 0; p < 3; ++p) f.t[p] = *reinterpret_cast<const uint4*>(blk + 256 * p + nat);
    return f;
  }
  static __device__ __forceinline__ void store(float* blk, const Frag& f, int nat) {
#pragma unroll
    for (int p = 0; p < 3; ++p) *reinterpret_cast<uint4*>(blk + 256 * p + nat) = f.t[p];
  }
  static __device__ __forceinline__ unsigned int neg2(unsigned int u) { return u ^ 0x80008000u; }
  static __device__ __forceinline__ floatx4 mm(const uint4& a, const uint4& b, floatx4 c) {
    typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf, a), __builtin_bit_cast(v8bf, b), c, 0, 0, 0);
  }
  // x.re += A B, x.im += A C over the six term products, small ones first
  static __device__ __forceinline__ void six(Acc& x, const Frag& A, const uint4 (&B)[3], const uint4 (&C)[3]) {
    constexpr int PA[6] = {1, 0, 2, 0, 1, 0}, PB[6] = {1, 2, 0, 1, 0, 0};
    Acc t = acc_zero();
#pragma unroll
    for (int p = 0; p < 6; ++p) {
      t.re = mm(A.t[PA[p]], B[PB[p]], t.re);
      t.im = mm(A.t[PA[p]], C[PB[p]], t.im);
    }
    x.re += t.re;
    x.im += t.im;
  }
  // Re(conj(q) p) = qr pr + qi pi, Im(conj(q) p) = qr pi - qi pr
  static __device__ __forceinline__ void pqh(Acc& x, const Frag& P, const Frag& Q) {
    uint4 C[3];
#pragma unroll
    for (int p = 0; p < 3; ++p) C[p] = make_uint4(P.t[p].z, P.t[p].w, neg2(P.t[p].x), neg2(P.t[p].y));
    six(x, Q, P.t, C);
  }
  // Re(q p) = qr pr - qi pi, Im(q p) = qr pi + qi pr
  static __device__ __forceinline__ void pq(Acc& x, const Frag& P, const Frag& Qt) {
    uint4 B[3], C[3];
#pragma unroll
    for (int p = 0; p < 3; ++p) {
      B[p] = make_uint4(P.t[p].x, P.t[p].y, neg2(P.t[p].z), neg2(P.t[p].w));
      C[p] = make_uint4(P.t[p].z, P.t[p].w, P.t[p].x, P.t[p].y);
    }
    six(x, Qt, B, C);
  }
};

// Keeps the compiler from computing what depends on a block's registers (its
// split terms) ahead of the loop that uses it, for all slots at once.
__device__ __forceinline__ void pin(Acc& a) { asm volatile("" : "+v"(a.re), "+v"(a.im)); }

__device__ __forceinline__ Acc acc_scale(const Acc& a, float s) {
  Acc b;
  b.re = a.re * s;
  b.im = a.im * s;
  return b;
}
__device__ __forceinline__ Acc acc_neg(const Acc& a) {
  Acc b;
  b.re = -a.re;
  b.im = -a.im;
  return b;
}

__device__ __forceinline__ double bcast64(double v, int lane) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffffLL), lane);
  const int hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// State of the in-wave factorisation and inversion of a 16 x 16 diagonal
// block.  CORR: the multipliers come from the rows of A, and the factor itself
// goes to LDS as well.
template <bool CORR>
struct Diag {
  static constexpr bool kCorr = CORR;
  Acc A;           // row m: columns > j of A, columns <= j of Y
  floatx4 cr, ci;  // columns 4 (j / 4) .. + 3 of A at row m, on every lane; with CORR the
                   // conjugates of rows 4 (j / 4) .. + 3 at column m instead
  float rs;        // 1 / d_j of the column to come
  float rsm;       // 1 / d_m
  int fail;
  double p64;      // FP64 Schur diagonal of row m (on the lane holding (m, m))
  float* rows;     // with CORR: LDS scratch of kBlk floats, 16-byte aligned
  float* keep;     // with CORR: kBlk floats of LDS that take the factor below its diagonal, zero
                   // elsewhere: real part of column j, row m at 16 j + m, imaginary part 256 further
  int m, q;
};

// v -= l * (row j of v) on every lane for the register pairs (re, im) of A
// and Y, l = lx + i ly: the row broadcast is a DPP operand of the FMA (the
// compiler folds DPP moves into multiplications but not into FMAs, and
// separate moves are a third of the column's instructions).  Per value the
// order is fma(-lx, b, fma(+-ly, b', v)).  The copies (c, e) of columns take
// part in the row update (STAP_COLS); copies of rows (STAP_ROWS) take c -=
// conj(l of that row) a, a = ax + i ay the lane's own copy of row j, in the
// same order, which gives them the bits of the rows that they copy.
// l is zero on row j itself, so the broadcast reads the row's old value
// whatever has been written, and every register's uses are at least 4
// instructions apart (DPP reads need two wait states after a write); the
// s_nops keep that distance to the compiler's instructions on both sides.
#define STAP_DPP(J) " row_newbcast:%[" J "] row_mask:0xf bank_mask:0xf\n"
#define STAP_F(D, S, L) "v_fmac_f32_dpp " D ", " S ", " L STAP_DPP("j")
#define STAP_ROWUPD(P) P("%[r0]", "%[i0]") P("%[r1]", "%[i1]") P("%[r2]", "%[i2]") P("%[r3]", "%[i3]")
#define STAP_P1(R, I) STAP_F(R, I, "%[ly]")
#define STAP_P2(R, I) STAP_F(I, "-" R, "%[ly]")
#define STAP_P3(R, I) STAP_F(R, "-" R, "%[lx]")
#define STAP_P4(R, I) STAP_F(I, "-" I, "%[lx]")
#define STAP_C1(N) "v_fmac_f32_dpp %[c" N "], -%[ly], %[ay]" STAP_DPP("j" N)
#define STAP_C2(N) "v_fmac_f32_dpp %[e" N "], %[ly], %[ax]" STAP_DPP("j" N)
#define STAP_C3(N) "v_fmac_f32_dpp %[c" N "], -%[lx], %[ax]" STAP_DPP("j" N)
#define STAP_C4(N) "v_fmac_f32_dpp %[e" N "], -%[lx], %[ay]" STAP_DPP("j" N)
#define STAP_ASM(C1, C2, C3, C4, ...)                                                                      \
  asm("s_nop 1\n" C1 STAP_ROWUPD(STAP_P1) C2 STAP_ROWUPD(STAP_P2) C3 STAP_ROWUPD(STAP_P3) C4               \
          STAP_ROWUPD(STAP_P4) "s_nop 1"                                                                   \
      : [r0] "+v"(ar0), [r1] "+v"(ar1), [r2] "+v"(ar2), [r3] "+v"(ar3), [i0] "+v"(ai0), [i1] "+v"(ai1),     \
        [i2] "+v"(ai2), [i3] "+v"(ai3), [c1] "+v"(cr1), [c2] "+v"(cr2), [c3] "+v"(cr3), [e1] "+v"(ci1),     \
        [e2] "+v"(ci2), [e3] "+v"(ci3)                                                                     \
      : [lx] "v"(lx), [ly] "v"(ly), [j] "n"(j), ##__VA_ARGS__)
#define STAP_COLS(C1, C2, C3, C4) STAP_ASM(C1, C2, C3, C4)
#define STAP_ROWS(C1, C2, C3, C4)                                                                          \
  STAP_ASM(C1, C2, C3, C4, [ax] "v"(ax), [ay] "v"(ay), [j1] "n"(4 * jq + 1), [j2] "n"(4 * jq + 2),          \
           [j3] "n"(4 * jq + 3))

// Column j of diag_factor_inv().  The inverse is formed in place: once the
// multipliers l_mj of column j are taken, A's column j is dead and Y's column
// j (X[m] = Y[m] / d_m, Y starts as the identity) comes to life in its
// registers, so one row update Y[m][c <= j], A[m][c > j] -= (l_mj / d_j) row j
// serves both; rows at or before j take none (l is zero there) and the lane
// of row j records 1 / d_j for the final scaling.  What is left above the
// diagonal at the end is dropped by diag_end().
//
// The multipliers of a column are read from a copy of the current four
// columns that every lane of a row keeps (cr, ci), updated like A itself and
// refreshed every fourth column: a cross-lane read through the LDS pipe, with
// its latency, once per four columns instead of once per column.
//
// With CORR the multipliers l_mj come from row j instead, as conj(A[j][m]): row
// and column of a Hermitian block drift apart in the rounding of the earlier
// columns, and products of a multiplier from the one and a row from the other
// magnify the difference by |l| / d (on clutter covariances the factor's
// backward error was up to 45 times that of products which agree, and the
// once-refined error 2 to 3 times: 96 DOF 8.1e-7, so 4.8e-7).  The copies are
// then of the current four rows, with their very bits, and below the diagonal
// A itself is never read.  Results that are not refined, and those of tuned
// shapes, keep the columns' rounding, which the systems' conditioning shows.
//
// The pivot is taken in FP64: every lane keeps, for its row m, p64 =
// (loaded diagonal R_mm) - (sum over earlier block columns of |L_mk|^2, FP64
// sums of the FP32 factor) - (sum over earlier columns of this block of
// |l_mk|^2, accumulated here in FP64), so d_j^2 = p64 of row j (read from the
// lane holding the block's diagonal element j) and the status test is
// p64 > 0 in FP64; the factorisation continues with d_j^2 rounded to FP32.
// There is no branch: after a non-positive pivot the remaining columns run
// on meaningless values and only the first failing index is kept, so the 16
// columns form one straight-line block the compiler can overlap.
template <int j, class S>
__device__ __forceinline__ void diag_pivot(S& s) {
  const double piv64 = bcast64(s.p64, j + 16 * (j >> 2));  // row j's FP64 Schur diagonal, wave-uniform
  s.fail = (s.fail == 0 && !(piv64 > 0.0)) ? j + 1 : s.fail;
  s.rs = __builtin_amdgcn_rsqf((float)piv64);
}
template <int j, class S>
__device__ __forceinline__ void diag_col(S& s) {
  constexpr int jq = j >> 2, ji = j & 3;
  if constexpr (ji == 0 && S::kCorr) {
    // all rows go out, which spares a mask; a wave's LDS accesses keep their order
    *reinterpret_cast<floatx4*>(s.rows + 16 * s.m + 4 * s.q) = s.A.re;
    *reinterpret_cast<floatx4*>(s.rows + 256 + 16 * s.m + 4 * s.q) = s.A.im;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      s.cr[i] = s.rows[16 * (4 * jq + i) + s.m];
      s.ci[i] = -s.rows[256 + 16 * (4 * jq + i) + s.m];
    }
  } else if constexpr (ji == 0) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      s.cr[i] = __shfl(s.A.re[i], s.m + 16 * jq);
      s.ci[i] = __shfl(s.A.im[i], s.m + 16 * jq);
    }
  }
  const float rs = s.rs, r2 = rs * rs;
  const float ax = s.m > j ? s.cr[ji] : 0.f, ay = s.m > j ? s.ci[ji] : 0.f;  // A[m][j] or conj(A[j][m])
  const float lx = ax * r2, ly = ay * r2;                                    // l_mj / d_j
  s.rsm = (s.m == j) ? rs : s.rsm;
  // l_mj in FP32, squared and summed in FP64 for row m
  const float lr = ax * rs, li = ay * rs;
  if constexpr (S::kCorr) {  // the four lanes of row m write the same
    s.keep[16 * j + s.m] = lr;
    s.keep[256 + 16 * j + s.m] = li;
  }
  s.p64 -= (double)lr * (double)lr + (double)li * (double)li;
  if constexpr (j < 15) diag_pivot<j + 1>(s);  // its latency passes behind the update
  s.A.re[ji] = s.q == jq ? (s.m == j ? 1.f : 0.f) : s.A.re[ji];
  s.A.im[ji] = s.q == jq ? 0.f : s.A.im[ji];
  float ar0 = s.A.re[0], ar1 = s.A.re[1], ar2 = s.A.re[2], ar3 = s.A.re[3];
  float ai0 = s.A.im[0], ai1 = s.A.im[1], ai2 = s.A.im[2], ai3 = s.A.im[3];
  float cr1 = s.cr[1], cr2 = s.cr[2], cr3 = s.cr[3], ci1 = s.ci[1], ci2 = s.ci[2], ci3 = s.ci[3];
  // A[m][c] -= l_mj conj(l_cj) = (A[m][j] / d_j^2) A[j][c], and Y likewise
  if constexpr (ji == 3)
    STAP_COLS("", "", "", "");
  else if constexpr (S::kCorr && ji == 0)
    STAP_ROWS(STAP_C1("1") STAP_C1("2") STAP_C1("3"), STAP_C2("1") STAP_C2("2") STAP_C2("3"),
              STAP_C3("1") STAP_C3("2") STAP_C3("3"), STAP_C4("1") STAP_C4("2") STAP_C4("3"));
  else if constexpr (S::kCorr && ji == 1)
    STAP_ROWS(STAP_C1("2") STAP_C1("3"), STAP_C2("2") STAP_C2("3"), STAP_C3("2") STAP_C3("3"),
              STAP_C4("2") STAP_C4("3"));
  else if constexpr (S::kCorr)
    STAP_ROWS(STAP_C1("3"), STAP_C2("3"), STAP_C3("3"), STAP_C4("3"));
  else if constexpr (ji == 0)
    STAP_COLS(STAP_P1("%[c1]", "%[e1]") STAP_P1("%[c2]", "%[e2]") STAP_P1("%[c3]", "%[e3]"),
              STAP_P2("%[c1]", "%[e1]") STAP_P2("%[c2]", "%[e2]") STAP_P2("%[c3]", "%[e3]"),
              STAP_P3("%[c1]", "%[e1]") STAP_P3("%[c2]", "%[e2]") STAP_P3("%[c3]", "%[e3]"),
              STAP_P4("%[c1]", "%[e1]") STAP_P4("%[c2]", "%[e2]") STAP_P4("%[c3]", "%[e3]"));
  else if constexpr (ji == 1)
    STAP_COLS(STAP_P1("%[c2]", "%[e2]") STAP_P1("%[c3]", "%[e3]"),
              STAP_P2("%[c2]", "%[e2]") STAP_P2("%[c3]", "%[e3]"),
              STAP_P3("%[c2]", "%[e2]") STAP_P3("%[c3]", "%[e3]"),
              STAP_P4("%[c2]", "%[e2]") STAP_P4("%[c3]", "%[e3]"));
  else
    STAP_COLS(STAP_P1("%[c3]", "%[e3]"), STAP_P2("%[c3]", "%[e3]"), STAP_P3("%[c3]", "%[e3]"),
              STAP_P4("%[c3]", "%[e3]"));
  s.A.re = floatx4{ar0, ar1, ar2, ar3};
  s.A.im = floatx4{ai0, ai1, ai2, ai3};
  s.cr = floatx4{s.cr[0], cr1, cr2, cr3};
  s.ci = floatx4{s.ci[0], ci1, ci2, ci3};
}
template <int j, class S>
__device__ __forceinline__ void diag_cols(S& s) {
  diag_col<j>(s);
  if constexpr (j < 15) diag_cols<j + 1>(s);
}
#undef STAP_DPP
#undef STAP_F
#undef STAP_ROWUPD
#undef STAP_P1
#undef STAP_P2
#undef STAP_P3
#undef STAP_P4
#undef STAP_C1
#undef STAP_C2
#undef STAP_C3
#undef STAP_C4
#undef STAP_ASM
#undef STAP_COLS
#undef STAP_ROWS

template <class S>
__device__ __forceinline__ void diag_begin(S& s, const Acc& A, double p64, float* rows = nullptr, float* keep = nullptr) {
  const int l = lane_tid() & 63;
  s.A = A;
  s.rows = rows;
  s.keep = keep;
  s.cr = s.ci = floatx4{0.f, 0.f, 0.f, 0.f};
  s.rsm = 1.f;
  s.fail = 0;
  s.p64 = p64;
  s.m = l & 15;
  s.q = l >> 4;
  diag_pivot<0>(s);
}
// SIGN / d_m times row m of Y, zero above the diagonal.
template <int SIGN, class S>
__device__ __forceinline__ Acc diag_end(const S& s) {
  const float sc = SIGN < 0 ? -s.rsm : s.rsm;
  Acc X;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const bool lower = 4 * s.q + i <= s.m;
    X.re[i] = lower ? s.A.re[i] * sc : 0.f;
    X.im[i] = lower ? s.A.im[i] * sc : 0.f;
  }
  return X;
}

// Factor the Hermitian 16 x 16 block A (full, both triangles; with CORR the
// upper one is read) as L L^H inside one wave and return X = SIGN L^-1 (lower
// triangular) and, with CORR, leave L in LDS at keep, but for its diagonal,
// which dm returns (row m's element on the lanes of row m).  Column j: pivot
// d_j = sqrt(A[j][j]) (taken in FP64 as above, p64 the lane's starting value
// for its row: loaded diagonal minus the earlier block columns), l_mj =
// A[m][j] / d_j for m > j, then A[m][c] -= l_mj conj(l_cj) for m, c > j; the
// inverse is accumulated as X <- L_j^-1 X with L_j the identity carrying
// column j of L (row j of X divided by d_j, then row m -= l_mj row j), the row
// divisions deferred.  conj(l_cj) is read as A[j][c] from row j, which lives in
// the same 16-lane row of the wave (a DPP broadcast).  Returns 0 or the 1-based
// index of the first non-positive pivot.  The wave runs at raised priority:
// the other waves of its system wait for it.
template <int SIGN, bool CORR>
__device__ __forceinline__ int diag_factor_inv(const Acc& A, Acc& X, float& dm, double p64, float* rows, float* keep) {
  Diag<CORR> s;
  diag_begin(s, A, p64, rows, keep);
  __builtin_amdgcn_s_setprio(3);
  diag_cols<0>(s);
  __builtin_amdgcn_s_setprio(0);
  X = diag_end<SIGN>(s);
  if (CORR) dm = 1.f / s.rsm;
  return s.fail;
}

// The lane's own diagonal element of a block in fragment order (lane (m, q)
// holds X[m][4q + i]; the element (m, m) sits in lane q = m / 4, register
// m % 4), or 0 on the other lanes.
__device__ __forceinline__ float blk_diag(const Acc& A) {
  const int l = lane_tid() & 63, m = l & 15, q = l >> 4;
  float v = 0.f;
#pragma unroll
  for (int i = 0; i < 4; ++i) v = (m == 4 * q + i) ? A.re[i] : v;
  return v;
}

// Row sums of |X|^2 of a block in fragment order, in FP64, on every lane of
// the row (lane (m, q) holds row m, columns 4q .. 4q + 3).
__device__ __forceinline__ double blk_row_norm2(const Acc& x) {
  double p = 0.0;
#pragma unroll
  for (int i = 0; i < 4; ++i)
    p += (double)x.re[i] * (double)x.re[i] + (double)x.im[i] * (double)x.im[i];
  p += __shfl_xor(p, 16);
  p += __shfl_xor(p, 32);
  return p;
}

// Level of refinement of a blocked solve: none, FP64 refinement, and FP64
// refinement with the corrected factorisation (rows' multipliers in the
// diagonal blocks, panels corrected for the error of the inverse).
constexpr int kPlain = 0, kRefined = 1, kCorrected = 2;

// Static layout of one system with NB block columns of R_L and NS block rows
// of steering vectors (both run-time), NW waves, and per wave NSL register
// slots for L blocks and NSM for M blocks (compile time).  L blocks are
// numbered column by column from the diagonal down, M blocks column by
// column, each set dealt round-robin to the waves (block g -> wave g % NW,
// slot g / NW).  The blocks still active at a step are a suffix of each
// order, so every step is balanced to within one block per wave and set.
// Loops over a wave's blocks run over its slots (unrolled, so register
// indices are constants) and test the slot's block coordinates, which are
// run-time values (wave-uniform).
template <int NSL_, int NSM_, int NW_>
struct BCfg {
  static constexpr int NSL = NSL_, NSM = NSM_, NW = NW_;
  static constexpr int NT = 64 * NW;
  // L and M slots per wave a (NB, NS) system needs
  __host__ __device__ static constexpr int lslots(int NB) { return (NB * (NB + 1) / 2 + NW - 1) / NW; }
  __host__ __device__ static constexpr int mslots(int NB, int NS) { return (NS * NB + NW - 1) / NW; }
  // Whether the blocks of L that the solves multiply by are split by their
  // owner, once, or by each of their users.  By the users the split is off
  // the path between two barriers; from three M blocks per wave on its
  // repetition costs more than that (256 bins x 64 blocks: 192 DOF, 48
  // steering vectors 21.99 ms per pass split by the users, 21.49 by the
  // owner; 96 DOF, 64 vectors, 128 x 32 systems 1078 and 1035 us; 96 DOF, 16
  // vectors 7.13 and 7.30 ms).
  static constexpr bool kOwnerSplits = NSM > 2;
  // LDS: exchange blocks (NB + NS + 1 for the factorisation, one more where
  // it is corrected; two times NB
  // blocks of L and NS for the solves; with refinement, all NS NB blocks
  // of Z in FP32 for the residual), the gamma
  // partials [NB][16 NS] (FP64), a flag, the FP64 row sums of |L|^2 over the
  // finished block columns [16 NB] and the loaded diagonal [16 NB] (for the
  // FP64 pivots)
  __host__ __device__ static constexpr size_t xbytes(int NB, int NS, int level) {
    const size_t kB = level ? OpSplit::kB : OpF32::kB;
    const size_t f = (NB + NS + (level == kCorrected ? 2 : 1)) * kB * 4, s = (2 * NB * (kOwnerSplits ? kB : kBlk) + NS * kB) * 4;
    const size_t z = level ? (size_t)NS * NB * kBlk * 4 : 0;
    return f > s ? (f > z ? f : z) : (s > z ? s : z);
  }
  __host__ __device__ static constexpr size_t lds_bytes(int NB, int NS, int level) {
    return xbytes(NB, NS, level) + (size_t)NB * 16 * NS * 8 + 16 + (size_t)NB * 16 * (8 + 4);
  }
};

// Block coordinates of a wave's register slots.
template <class C>
struct Slots {
  int NB, NS;
  bool lv[C::NSL], mv[C::NSM];
  int lr[C::NSL], lc[C::NSL], mr[C::NSM], mc[C::NSM];
  __device__ __forceinline__ Slots(int D, int S, int wave) {
    NB = (D + 15) >> 4;
    NS = (S + 15) >> 4;
#pragma unroll
    for (int t = 0; t < C::NSL; ++t) {
      const int g = wave + C::NW * t;
      lv[t] = false;
      lr[t] = lc[t] = 0;
      int start = 0;
      for (int J = 0; J < NB; ++J) {
        const int len = NB - J;
        if (g >= start && g < start + len) {
          lv[t] = true;
          lc[t] = J;
          lr[t] = J + (g - start);
        }
        start += len;
      }
    }
#pragma unroll
    for (int t = 0; t < C::NSM; ++t) {
      const int g = wave + C::NW * t;
      mv[t] = g < NS * NB;
      mc[t] = g / NS;
      mr[t] = g - (g / NS) * NS;
    }
  }
};
// Number of L block (I, J) in that order.
__device__ __forceinline__ int lblock(int NB, int I, int J) { return J * NB - J * (J - 1) / 2 + (I - J); }

// The LDS regions of a system (lds_bytes(NB, NS, LEVEL) at xlds).
template <class C, int LEVEL>
struct SolveLds {
  typedef std::conditional_t<LEVEL != kPlain, OpSplit, OpF32> Op;
  float* xb;      // exchange blocks
  float* dinv;    // minus the inverse of the current diagonal block's factor
  float* diag;    // that factor (kCorrected)
  double* gpart;  // gamma partials
  int* sflag;     // pivot status
  double* d64;    // FP64 row sums of |L|^2
  float* rdiag;   // loaded diagonal
  __device__ __forceinline__ SolveLds(unsigned char* xlds, int NB, int NS) {
    xb = reinterpret_cast<float*>(xlds);
    dinv = xb + (size_t)(NB + NS) * Op::kB;
    diag = dinv + Op::kB;
    gpart = reinterpret_cast<double*>(xlds + C::xbytes(NB, NS, LEVEL));
    sflag = reinterpret_cast<int*>(gpart + NB * 16 * NS);
    d64 = reinterpret_cast<double*>(reinterpret_cast<unsigned char*>(sflag) + 16);
    rdiag = reinterpret_cast<float*>(d64 + NB * 16);
  }
};

__device__ __forceinline__ doublex4 mfma64(double a, double b, doublex4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// Whether rows of D complex elements starting at p keep 16-byte alignment
// at every even column.
__device__ __forceinline__ bool rows16(const void* p, int D) {
  return (D & 1) == 0 && (reinterpret_cast<uintptr_t>(p) & 15) == 0;
}
// Elements k .. k+3 of row s of a [rows][D] array (k a multiple of 4), zero
// from column D on and for rows not in the array; two 16-byte loads where
// the rows allow it (vec = rows16()), which fetches a lane's 32 bytes in one
// go.  The element index passes through an empty asm statement, so that the
// compiler neither merges the loads with an earlier read of the same
// elements (keeping those live across the solve costs more registers than
// reading them again from the cache) nor, as volatile loads would be, issues
// them one round trip at a time.
__device__ __forceinline__ void load4(const float2* base, int s, int k, bool row_ok, int D, bool vec, float2 (&v)[4]) {
  int o = s * D + k;
  asm volatile("" : "+v"(o));
  if (vec && row_ok && k + 4 <= D) {
    const float4 a = *reinterpret_cast<const float4*>(base + o);
    const float4 b = *reinterpret_cast<const float4*>(base + o + 2);
    v[0] = make_float2(a.x, a.y);
    v[1] = make_float2(a.z, a.w);
    v[2] = make_float2(b.x, b.y);
    v[3] = make_float2(b.z, b.w);
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = (row_ok && k + i < D) ? base[o + i] : make_float2(0.f, 0.f);
  }
}
__device__ __forceinline__ void store4(float2* base, int s, int k, bool row_ok, int D, bool vec, const float2 (&v)[4]) {
  const int o = s * D + k;
  if (vec && row_ok && k + 4 <= D) {
    *reinterpret_cast<float4*>(base + o) = make_float4(v[0].x, v[0].y, v[1].x, v[1].y);
    *reinterpret_cast<float4*>(base + o + 2) = make_float4(v[2].x, v[2].y, v[3].x, v[3].y);
  } else if (row_ok) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (k + i < D) base[o + i] = v[i];
  }
}

// -M = -V^H blocks of the wave's slots (zero beyond S and D).
template <class C>
__device__ __forceinline__ void load_steer(const Slots<C>& sl, const float2* __restrict__ steer, int D, int S,
                                           Acc (&am)[C::NSM]) {
  const int l = lane_tid() & 63, m = l & 15, q = l >> 4;
  const bool vec = rows16(steer, D);
#pragma unroll
  for (int t = 0; t < C::NSM; ++t) {
    Acc a = acc_zero();
    if (sl.mv[t]) {
      const int s = 16 * sl.mr[t] + m;
      float2 v[4];
      load4(steer, s, 16 * sl.mc[t] + 4 * q, s < S, D, vec, v);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        a.re[i] = -v[i].x;
        a.im[i] = v[i].y;
      }
    }
    am[t] = a;
  }
}

// With refinement a system is solved as 4^-k R_L, k such that its diagonal is
// about 1: the solution then stays in the range of the split's low terms (from
// 2^-110) and of the pivots' square roots (from 2^-126) for any R_L (96 DOF, 64
// vectors, elements of 4e37: error 2.7e-6 without, 5.0e-8 with; of 1e-33 four
// systems of 128 failed).  A power of 4 keeps every bit otherwise: weights come
// out 2^k times too large and are scaled back as they are written.
struct SysScale {
  float r, w;  // 4^-k, 2^-k
  __device__ __forceinline__ explicit SysScale(float diag) {
    const int e = (int)((__float_as_uint(diag) >> 23) & 0xffu) - 127;  // 128: not finite
    int k = diag > 0.f && e < 128 ? max(e, -126) >> 1 : 0;
    k = __builtin_amdgcn_readfirstlane(k);
    r = __uint_as_float((unsigned int)(127 - 2 * k) << 23);
    w = __uint_as_float((unsigned int)(127 - k) << 23);
  }
};

// Solve one system (D <= 16 NB, S <= 16 NS, lslots(NB) <= NSL,
// mslots(NB, NS) <= NSM).  al holds the wave's blocks of minus the loaded
// covariance (identity beyond D, diagonal blocks with both triangles), with
// refinement times sc.r, am those of -M: blocks still to be finished are kept
// negated, so that every update adds (x -= P Q^H is -x += P Q^H) and the panel
// product with -Linv_JJ restores the sign, all exactly.  L.rdiag holds the
// loaded diagonal of the diagonal blocks, unscaled (written by the wave that
// owns them), and L.d64 zeros, visible after the
// next barrier.  With refinement src.get(J, I) yields, on lane (m, q), R_L[16J +
// 4q + s][16I + m], s = 0..3; it must stay readable for the whole call.  W is
// this system's [S][D] output, info its status word (may be null).  park
// (may be null) is LDS of at least NS NB blocks that is free once the last
// residual has been formed (the source, when it lives in LDS): the last
// refinement step keeps u there instead of in W.
template <class C, int LEVEL, class RSrc>
__device__ __forceinline__ void bsolve_blocks(const Slots<C>& sl, Acc (&al)[C::NSL], Acc (&am)[C::NSM],
                                              const SolveLds<C, LEVEL>& L, const RSrc& src,
                                              const float2* __restrict__ steer, float2* __restrict__ W,
                                              int* __restrict__ info, const Dims& d, float* park, SysScale sc) {
  constexpr bool REFINE = LEVEL != kPlain, CORR = LEVEL == kCorrected;
  typedef typename SolveLds<C, LEVEL>::Op Op;
  typedef typename Op::Frag Frag;
  constexpr int NSL = C::NSL, NSM = C::NSM, kB = Op::kB;
  const int D = d.D, S = d.S, NB = sl.NB, NS = sl.NS;
  float* const xb = L.xb;
  const int tid = lane_tid(), lane = tid & 63, m = lane & 15, q = lane >> 4;
  const int nat = nat_ofs();

  // ---- factorisation with the forward solve of the steering rows.  The
  // wave owning diagonal block J+1 applies its last update (from column J)
  // first and factors it right away, while the other waves finish the
  // updates of step J; step J = -1 only factors diagonal block 0.
  int fail = 0;
  for (int J = -1; J < NB; ++J) {
    if (J >= 0) {
      __syncthreads();
      fail = *L.sflag;
      if (fail) break;
      const Frag Q = Op::load(L.dinv, nat);
#pragma unroll
      for (int t = 0; t < NSL; ++t) {
        if (sl.lv[t] && sl.lc[t] == J && sl.lr[t] != J) {
          Acc x = acc_zero();
          Op::pqh(x, Op::frag(al[t]), Q);
          if (CORR) {
            // X = A Linv^H carries the inverse's error, |L| |Linv| times that
            // of a substitution, into everything that follows; one step of
            // X += (A - X L^H) Linv^H takes it out (96 DOF 4.8e-7, so 7e-8
            // to 1.1e-7; 5 to 9 % of the solve)
            Acc e = al[t];
            Op::pqh(e, Op::frag(x), Op::load(L.diag, nat));
            Op::pqh(x, Op::frag(e), Q);
          }
          al[t] = x;
          Op::store(xb + sl.lr[t] * kB, Op::frag(x), nat);
          // FP64 row sums of |L|^2 for the pivots of block row lr (one
          // panel block per block row and step: no other writer)
          const double pn = blk_row_norm2(x);
          if (q == 0) L.d64[16 * sl.lr[t] + m] += pn;
        }
      }
#pragma unroll
      for (int t = 0; t < NSM; ++t) {
        if (sl.mv[t] && sl.mc[t] == J) {
          Acc x = acc_zero();
          Op::pqh(x, Op::frag(am[t]), Q);
          am[t] = x;
          Op::store(xb + (NB + sl.mr[t]) * kB, Op::frag(x), nat);
        }
      }
      __syncthreads();
    }
    int tn = -1;
#pragma unroll
    for (int t = 0; t < NSL; ++t)
      if (J + 1 < NB && sl.lv[t] && sl.lr[t] == J + 1 && sl.lc[t] == J + 1) tn = t;
    if (tn >= 0) {
      // the diagonal code exists once: the slot's block is copied in and out
      Acc A = acc_zero();
#pragma unroll
      for (int t = 0; t < NSL; ++t)
        if (tn == t) {
          A.re = al[t].re;
          A.im = al[t].im;
        }
      if (J >= 0) {
        const Frag P = Op::load(xb + (J + 1) * kB, nat);
        Op::pqh(A, P, P);
      }
      const int r = 16 * (J + 1) + m;
      const double p64 = (double)(REFINE ? L.rdiag[r] * sc.r : L.rdiag[r]) - (J >= 0 ? L.d64[r] : 0.0);
      Acc X;
      float dm = 0.f;
      const int f = diag_factor_inv<-1, CORR>(acc_neg(A), X, dm, p64, L.dinv, L.diag);
      Op::store(L.dinv, Op::frag(X), nat);
      if (CORR) {
        Acc F;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int c = 4 * q + i;
          F.re[i] = c == m ? dm : L.diag[16 * c + m];
          F.im[i] = L.diag[256 + 16 * c + m];
        }
        Op::store(L.diag, Op::frag(F), nat);
      }
#pragma unroll
      for (int t = 0; t < NSL; ++t)
        if (tn == t) {
          al[t].re = X.re;
          al[t].im = X.im;
        }
      if (lane == 0) *L.sflag = f ? 16 * (J + 1) + f : 0;
    }
    if (J >= 0) {
#pragma unroll
      for (int t = 0; t < NSL; ++t)
        if (sl.lv[t] && sl.lc[t] > J && t != tn)
          Op::pqh(al[t], Op::load(xb + sl.lr[t] * kB, nat), Op::load(xb + sl.lc[t] * kB, nat));
#pragma unroll
      for (int t = 0; t < NSM; ++t)
        if (sl.mv[t] && sl.mc[t] > J)
          Op::pqh(am[t], Op::load(xb + (NB + sl.mr[t]) * kB, nat), Op::load(xb + sl.mc[t] * kB, nat));
    }
  }

  if (fail) {
    for (int e = tid; e < S * D; e += C::NT) W[e] = make_float2(0.f, 0.f);
    if (tid == 0 && info) *info = fail;
    return;
  }

  // ---- gamma_s = ||y_s||^2 (no refinement), partial per block column
  if (!REFINE || d.refine == 0) {
#pragma unroll
    for (int t = 0; t < NSM; ++t) {
      if (sl.mv[t]) {
        float p = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) p = fmaf(am[t].re[i], am[t].re[i], fmaf(am[t].im[i], am[t].im[i], p));
        p += __shfl_xor(p, 16);
        p += __shfl_xor(p, 32);
        if (q == 0) L.gpart[sl.mc[t] * 16 * NS + 16 * sl.mr[t] + m] = p;
      }
    }
  }

  // ---- triangular solves with the stored factor.  The blocks of L that a
  // step multiplies by pass through LDS, two steps' worth in turn: a step's
  // products run while the owners put the next step's blocks into the other
  // half, so a step has two barriers.
  constexpr bool kOwner = C::kOwnerSplits && kB != kBlk;
  constexpr int kL = kOwner ? kB : kBlk;
  float* const zb = xb + (size_t)2 * NB * kL;
  auto half = [&](int J, int I) { return xb + (size_t)((J & 1) * NB + I) * kL; };
  auto l_frag = [&](int J, int I) { return kOwner ? Op::load(half(J, I), nat) : Op::frag(blk_load(half(J, I), nat)); };
  // Back solve, row form Z L = Y^H (M holds Y^H on entry, Z on exit).
  auto back_solve = [&]() {
    auto publish = [&](int J) {  // L_JI^T at I (-Linv_JJ^T at I = J)
#pragma unroll
      for (int t = 0; t < NSL; ++t)
        if (sl.lv[t] && sl.lr[t] == J) {
          float* const b = half(J, sl.lc[t]);
          blk_store_t(b, al[t]);
          if (kOwner) Op::store(b, Op::frag(blk_load(b, nat)), nat);
        }
    };
#pragma unroll
    for (int t = 0; t < NSM; ++t) am[t] = acc_neg(am[t]);
    __syncthreads();  // earlier readers of the exchange blocks are done
    publish(NB - 1);
    for (int J = NB - 1; J >= 0; --J) {
      __syncthreads();  // row J is there; the updates of step J + 1 are done
#pragma unroll
      for (int t = 0; t < NSM; ++t) {
        if (sl.mv[t] && sl.mc[t] == J) {
          Acc x = acc_zero();
          Op::pq(x, Op::frag(am[t]), l_frag(J, J));
          am[t] = x;
          if (J > 0) Op::store(zb + sl.mr[t] * kB, Op::frag(x), nat);
        }
      }
      if (J > 0) {
        publish(J - 1);
        __syncthreads();
#pragma unroll
        for (int t = 0; t < NSM; ++t)
          if (sl.mv[t] && sl.mc[t] < J)
            Op::pq(am[t], Op::load(zb + sl.mr[t] * kB, nat), l_frag(J, sl.mc[t]));
      }
    }
  };
  // Forward solve Y^H L^H = M (M negated on entry, Y^H on exit).
  auto forward_solve = [&]() {
    auto publish = [&](int J) {  // column J of L (-Linv_JJ at the diagonal)
#pragma unroll
      for (int t = 0; t < NSL; ++t)
        if (sl.lv[t] && sl.lc[t] == J) {
          pin(al[t]);
          if (kOwner) Op::store(half(J, sl.lr[t]), Op::frag(al[t]), nat);
          else blk_store(half(J, sl.lr[t]), al[t], nat);
        }
    };
    __syncthreads();
    publish(0);
    for (int J = 0; J < NB; ++J) {
      __syncthreads();
#pragma unroll
      for (int t = 0; t < NSM; ++t) {
        if (sl.mv[t] && sl.mc[t] == J) {
          Acc x = acc_zero();
          Op::pqh(x, Op::frag(am[t]), l_frag(J, J));
          am[t] = x;
          if (J + 1 < NB) Op::store(zb + sl.mr[t] * kB, Op::frag(x), nat);
        }
      }
      if (J + 1 < NB) {
        publish(J + 1);
        __syncthreads();
#pragma unroll
        for (int t = 0; t < NSM; ++t)
          if (sl.mv[t] && sl.mc[t] > J)
            Op::pqh(am[t], Op::load(zb + sl.mr[t] * kB, nat), l_frag(J, sl.mc[t]));
      }
    }
  };
  back_solve();

  const bool vecW = rows16(W, D), vecV = rows16(steer, D);
  if (REFINE) {
    for (int it = 0; it < d.refine; ++it) {
      const bool lds_park = park != nullptr && it == d.refine - 1;
      // keep the current u = conj(Z) in W (this lane's own elements; read
      // back by the same lane after the correction), or in park
#pragma unroll
      for (int t = 0; t < NSM; ++t) {
        if (sl.mv[t] && !lds_park) {
          const int s = 16 * sl.mr[t] + m;
          float2 u[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) u[i] = make_float2(am[t].re[i], -am[t].im[i]);
          store4(W, s, 16 * sl.mc[t] + 4 * q, s < S, D, vecW, u);
        }
      }
      // residual in row form: conj(r) = conj(v) - Z R_L, FP64 MFMA (FP32
      // operands converted exactly).  Every Z block is published; each M
      // block's owner sums over J.  Each complex product q p takes three real
      // products (Gauss): a1 += qr pr, a2 += qi pi, a3 += (qr + qi)(pr + pi),
      // then Re = a1 - a2 and Im = a3 - a1 - a2 (the FP64 sums qr + qi and
      // pr + pi of FP32 values are exact).  Lane (m, q) register i of an
      // accumulator holds column q + 4i of the block.
      __syncthreads();
#pragma unroll
      for (int t = 0; t < NSM; ++t)
        if (sl.mv[t]) blk_store(xb + (sl.mr[t] * NB + sl.mc[t]) * kBlk, am[t], nat);
      __syncthreads();
#pragma unroll
      for (int t = 0; t < NSM; ++t) {
        if (sl.mv[t]) {
          doublex4 a1 = {0.0, 0.0, 0.0, 0.0}, a2 = a1, a3 = a1;
          const float* zrow = xb + sl.mr[t] * NB * kBlk;
#pragma unroll 1
          for (int J = 0; J < NB; ++J) {
            const Acc z = blk_load(zrow + J * kBlk, nat);  // Z_{N,J}[m][4q + s]
            const Acc r = src.get(J, sl.mc[t], nat);
#pragma unroll
            for (int s4 = 0; s4 < 4; ++s4) {
              const double qr = r.re[s4], qi = r.im[s4], pr = z.re[s4], pi = z.im[s4];
              a1 = mfma64(qr, pr, a1);
              a2 = mfma64(qi, pi, a2);
              a3 = mfma64(qr + qi, pr + pi, a3);
            }
          }
          const doublex4 cr = (a1 - a2) * (double)sc.r, ci = (a3 - a1 - a2) * (double)sc.r;
          const int s = 16 * sl.mr[t] + m;
          // the slot's Z is in LDS now: its registers hold minus the
          // residual, column q + 4i in register i
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int k = 16 * sl.mc[t] + q + 4 * i;
            int o = s * D + k;
            asm volatile("" : "+v"(o));
            const float2 v = (s < S && k < D) ? steer[o] : make_float2(0.f, 0.f);
            am[t].re[i] = (float)(cr[i] - (double)v.x);
            am[t].im[i] = (float)((double)v.y + ci[i]);
          }
        }
      }
      __syncthreads();  // every Z block has been read
      // conj(r) rounded to FP32, back into fragment order through the
      // block's own (now free) Z position, or through its park slot, which
      // then takes the Z block itself (u for the correction)
#pragma unroll
      for (int t = 0; t < NSM; ++t) {
        if (sl.mv[t]) {
          float* zb = xb + (sl.mr[t] * NB + sl.mc[t]) * kBlk;
          float* tb = lds_park ? park + (sl.mr[t] * NB + sl.mc[t]) * kBlk : zb;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int o = bofs(m, q + 4 * i);
            tb[o] = am[t].re[i];
            tb[256 + o] = am[t].im[i];
          }
          am[t] = blk_load(tb, nat);
          if (lds_park) blk_store(tb, blk_load(zb, nat), nat);
        }
      }
      forward_solve();  // Y^H L^H = r^H
      back_solve();
      // Z += the correction (u kept in W or park)
#pragma unroll
      for (int t = 0; t < NSM; ++t) {
        if (sl.mv[t] && lds_park) {
          const Acc z = blk_load(park + (sl.mr[t] * NB + sl.mc[t]) * kBlk, nat);
          am[t].re += z.re;
          am[t].im += z.im;
        } else if (sl.mv[t]) {
          const int s = 16 * sl.mr[t] + m;
          float2 u[4];
          load4(W, s, 16 * sl.mc[t] + 4 * q, s < S, D, vecW, u);
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            am[t].re[i] += u[i].x;
            am[t].im[i] -= u[i].y;
          }
        }
      }
    }
    if (d.refine > 0) {
      // gamma_s = Re(v_s^H u_s) in FP64 for the refined u, u = conj(Z)
#pragma unroll
      for (int t = 0; t < NSM; ++t) {
        if (sl.mv[t]) {
          const int s = 16 * sl.mr[t] + m;
          float2 v[4];
          load4(steer, s, 16 * sl.mc[t] + 4 * q, s < S, D, vecV, v);
          double p = 0.0;
#pragma unroll
          for (int i = 0; i < 4; ++i)  // Re(conj(v) conj(z))
            p += (double)v[i].x * am[t].re[i] - (double)v[i].y * am[t].im[i];
          p += __shfl_xor(p, 16);
          p += __shfl_xor(p, 32);
          if (q == 0) L.gpart[sl.mc[t] * 16 * NS + 16 * sl.mr[t] + m] = p;
        }
      }
    }
  }
  __syncthreads();  // gamma partials

  // ---- w_s = u_s / sqrt(gamma_s), u_s = conj(z_s)
#pragma unroll
  for (int t = 0; t < NSM; ++t) {
    if (sl.mv[t]) {
      const int s = 16 * sl.mr[t] + m;
      double gam = 0.0;
      for (int J = 0; J < NB; ++J) gam += L.gpart[J * 16 * NS + s];
      const float g = REFINE ? 1.f / sqrtf((float)gam) * sc.w : 1.f / sqrtf((float)gam);
      float2 w[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) w[i] = make_float2(am[t].re[i] * g, -am[t].im[i] * g);
      store4(W, s, 16 * sl.mc[t] + 4 * q, s < S, D, vecW, w);
    }
  }
  if (tid == 0 && info) *info = 0;
}

}  // namespace stap
