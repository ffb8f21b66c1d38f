// The fused SQP iteration for one trajectory-optimisation solve per workgroup.
//
// One workgroup of up to kBlock threads owns one solve and runs whole SQP iterations
// (Algorithm 1) without returning to the host. Knot k of the solve is handled
// by a group of G lanes (G = 16 for 5..7 DoF, 8 for fewer), so a wavefront
// holds 64/G knots. Per iteration:
//   1. LQ (Sec. III-A, Eq. (1)): a thread per knot and half evaluates forward
//      dynamics (the inertia matrix's Cholesky factor; the bias forces) and shares
//      it through LDS; lane d of the knot's group then forms column d of the
//      dynamics Jacobian with one dual-number RNEA pass. Defects, gradients and the
//      current merit follow.
//   2. Schur complement (Eqs. (5)-(6)): lane j forms row j of theta_{k-1} and
//      entry j of gamma~ in FP64, then the group inverts the diagonal block by
//      Gauss-Jordan elimination (SPD, no pivoting).
//   3. Stair preconditioner (Eq. (6)): the FP64 variants apply it factored,
//      P v = D^-1 (v - O D^-1 v) with O the off-diagonal blocks of S~, so only
//      the rows of D^-1 are kept, and take the S~ product of the result from the
//      same two half-sweeps (pcg_half_sweeps, pcg_long); the all-FP32 variant's
//      lanes of knot k+1 form
//      the off-diagonal block -D_{k+1}^-1 phi_k D_k^-1 once and knot k reads
//      its transpose. The paper's single grid-wide synchronisation becomes a
//      workgroup barrier.
//   4. PCG on S~ lambda = gamma~ (Sec. II-B, III-B) in the pipelined
//      arrangement: the inner products of an iteration are reduced together
//      and share a barrier with the vector exchange, so an iteration needs two
//      workgroup barriers. Rows of S~ and P stay in registers; vectors are
//      exchanged through LDS. (The task-space variant and four knots per lane
//      group take the sums behind a barrier of their own; the all-FP32 variant
//      runs the standard arrangement.)
//   5. Step dZ = -G^-1 (g - C^T lambda) (Eq. (4)).
//   6. Line search (Eqs. (3), (7)): thread (alpha, knot) evaluates one trial
//      knot, or one thread each half of its dynamics; a fixed-order reduction
//      gives each candidate's merit.
// The Schur rows, gamma~, the block inverses, the PCG vectors and its inner
// products use Real (double; float for the all-FP32 variant). Dynamics and the
// line search's trial points use float; the explicit preconditioner blocks of
// the all-FP32 variant too.
//
// Task-space variant (TS): a tip tracking term 1/2 |p(q_k) - pref_k|^2_W per
// knot makes the joint block of Q_k dense, H_k = diag(Q_q + rho) + J^T W J
// (Gauss-Newton). Phase 1 then also factors H_k = L_k L_k^T and rewrites the
// QP in the variables y_k = T_k^-1 x_k, T_k = blkdiag(L_k^-T, I), whose state
// Hessian is diagonal again: A_k -> T_{k+1}^-1 A_k T_k, e_k -> T_{k+1}^-1 e_k,
// q_k -> T_k^T q_k, c_0 -> T_0^-1 c_0 (B_k is unchanged, its joint rows are
// zero). The Schur complement of the rewritten QP is congruent to that of
// Eq. (5) under blkdiag(T_k^-1), and so is the stair preconditioner of
// Eq. (6), so PCG takes the same iterates (multipliers scaled by T_k^T) and
// the same stopping value as on the dense-Q_k system; phases 2-4 run
// unchanged, and phase 5 maps the step and the multipliers back.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>
#include <utility>

#include "gato_internal.hpp"

namespace gato {

template <int ND>
struct Shape {
  static constexpr int NX = 2 * ND;
  static constexpr int NU = ND;
  static constexpr int G = (2 * ND > 8) ? 16 : 8;  // lanes per knot (power of two >= NX)
  static constexpr int SLOTS = kBlock / G;          // knots handled at once
  static constexpr int NL = ND * (ND + 1) / 2;      // packed Cholesky factor
};

// The FP64 variants run the PCG of pcg_half_sweeps (below).
template <class Real, int KPT>
constexpr bool half_sweeps() {
  return sizeof(Real) == 8;
}
// Four knots per lane group: the registers hold the D^-1 rows only, the A blocks
// stay in LDS (their velocity rows in FP32; the joint rows are [I, hI] by
// construction of the Euler step).
template <class Real, int KPT>
constexpr bool long_form() {
  return half_sweeps<Real, KPT>() && KPT == 4;
}
// Its vectors: knot k at row k + 1, zero rows beyond both ends. (K = 0: unused.)
template <int ND, int K>
struct PcgBufs {
  static constexpr int KH = K * Shape<ND>::SLOTS + 2;
  double z[KH][Shape<ND>::G];
  double v[KH][Shape<ND>::G];
  alignas(16) double red[128];   // per wavefront: four partial sums of each of two values, interleaved;
                                 // [64, 128): written by the lanes without one, never read
};

// QP blocks live in LDS when the workgroup holds at most 32 knots, or one knot
// per lane group, and with FP64 Schur rows also at two knots per lane group (but
// for the 6-7 DoF tip tracking variants, whose factors take that space); in the
// solve's global workspace otherwise. (7 DoF N = 64, 256 solves: Schur rows 13.6 ->
// 10.1 us and step 7.7 -> 3.5 us per SQP iteration.)
template <int ND, int KPT, class Real, bool TS>
struct BlockStore {
  static constexpr int KN = KPT * Shape<ND>::SLOTS;
  static constexpr bool kLds = (KPT == 1) || (KN <= 32) || (KPT == 2 && sizeof(Real) == 8 && !(TS && ND > 3));
  static constexpr int LB = kLds ? KN : 1;
};

// LDS that only some phases use: dynamics (qdd, Lf), line search (mp) and PCG
// (pcg; tv). The long form lets them share their space.
template <int ND, int KPT, class Real, bool LONG = long_form<Real, KPT>()>
struct PhaseSmem {
  using Sh = Shape<ND>;
  static constexpr int KN = KPT * Sh::SLOTS;
  static constexpr bool kHalf = half_sweeps<Real, KPT>();
  static constexpr int KV = kHalf ? 1 : KN;   // vectors of the other arrangements
  float qdd[KN][8];        // forward dynamics at the knot
  float Lf[KN][Sh::NL];    // packed Cholesky factor of the inertia matrix
  PcgBufs<ND, kHalf ? KPT : 0> pcg;
  union {
    double mp[kMaxAlpha][KN];  // per-knot merit terms of the step candidates (line search)
    Real tv[KV][Sh::G];        // exchange inside a lane group (PCG preconditioner)
  };
};
template <int ND, int KPT, class Real>
struct PhaseSmem<ND, KPT, Real, true> {
  using Sh = Shape<ND>;
  static constexpr int KN = KPT * Sh::SLOTS;
  static constexpr int KV = 1;
  union {
    struct {
      float qdd[KN][8];
      float Lf[KN][Sh::NL];
      double mp[kMaxAlpha][KN];
    };
    PcgBufs<ND, KPT> pcg;
  };
  Real tv[1][Sh::G];
  float Av[KN][ND][2 * ND];   // velocity rows of A_k
};

template <int ND, int KPT, class Real, bool TS>
struct Smem : PhaseSmem<ND, KPT, Real> {
  using Sh = Shape<ND>;
  static constexpr int G = Sh::G;
  static constexpr int NX = Sh::NX, NU = Sh::NU;
  static constexpr int KN = KPT * Sh::SLOTS;
  using BS = BlockStore<ND, KPT, Real, TS>;
  static constexpr bool kHalf = half_sweeps<Real, KPT>();
  static constexpr int KV = PhaseSmem<ND, KPT, Real>::KV;
  static constexpr int LP = kHalf ? 1 : BS::LB;
  float X[KN][G];          // iterate
  float U[KN][8];
  float dX[KN][G];         // step
  float dU[KN][8];
  float e[KN][G];          // defects e_k = f(x_k, u_k) - x_{k+1}
  float qg[KN][G];         // state gradients q_k
  float rg[KN][8];         // control gradients r_k
  double lam[kHalf ? KN : 1][G];   // multipliers between the PCGs
  Real rv[KV][G];          // PCG residual, shared for the preconditioner
  Real gv[KV][G];          // gamma~, shared for the reference norm
  Real pv[KV][G];          // vector shared for the S~ product
  Real sv[KV][G];          // Q_k^-1 times pv
  double piv[Sh::SLOTS][G];  // Gauss-Jordan pivot rows, one per lane group
  double red[2][3][kBlock / 64];  // per-wavefront partial sums
  double mp0[KN];          // per-knot merit terms at the current point
  double Qi[G], Qni[G];    // 1 / (Q + rho), 1 / (Q_N + rho) for the current rho
  double merit[kMaxAlpha + 1];
  float alpha[kMaxAlpha];
  float xs[G], xg[G], c0[G];
  int bad[2];              // per-iteration flag, indexed by iteration parity
  int xfail, xpad[3];      // split solve: a wait for another part gave up (16 bytes: keeps
                           // the blocks below 16-byte aligned for 128-bit LDS reads)
  float A[BS::LB][NX * NX];    // A_k
  float B[BS::LB][NX * NU];    // B_k
  float Dinv[LP][NX * NX]; // inverse diagonal blocks of S~
  float Poff[LP][NX * NX]; // P_{k+1,k}
};

// LDS of the task-space variant, placed after Smem.
template <int ND, int KPT>
struct TsSmem {
  static constexpr int KN = KPT * Shape<ND>::SLOTS;
  static constexpr int NL = Shape<ND>::NL;
  double Lc[KN][NL];     // Cholesky factor L_k of the joint block H_k (packed rows)
  double Li[KN][NL];     // L_k^-1 (packed rows)
  double tq[KN][8];      // joint-block vectors exchanged inside a lane group
  double mt[KN];         // tip tracking cost of each knot at the current iterate
  float Jt[KN][3][8];    // tip Jacobian J_k (column per joint)
  float pr[KN][4];       // reference tip positions
  float pe[KN][4];       // p(q_k) - pref_k at the current iterate
};

template <int ND, int KPT, class Real>
constexpr size_t ts_offset() {
  return (sizeof(Smem<ND, KPT, Real, true>) + 15) & ~(size_t)15;
}
template <int ND, int KPT, class Real, bool TS>
constexpr size_t smem_bytes() {
  return TS ? ts_offset<ND, KPT, Real>() + sizeof(TsSmem<ND, KPT>) : sizeof(Smem<ND, KPT, Real, false>);
}

// Packed lower-triangular storage, row i holding columns 0..i.
__device__ __forceinline__ constexpr int tri(int i, int j) { return i * (i + 1) / 2 + j; }

__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ---- Cross-lane sums. Every lane ends with the bit-identical total.
// The in-row patterns (quad permutations, row mirrors) read a valid lane for
// every lane, so those moves need no previous destination value; the row
// broadcasts that combine the four rows stay in registers (no LDS round trip).
template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xF, 0xF, true));
}
template <int CTRL>
__device__ __forceinline__ double dpp(double v) {
  const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xF, 0xF, true);
  return __hiloint2double(hi, lo);
}
// Row broadcasts (row_bcast:15 = 0x142, row_bcast:31 = 0x143) into the rows
// of ROWS; the other rows read 0.
template <int CTRL, int ROWS>
__device__ __forceinline__ float bcast(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, ROWS, 0xF, false));
}
template <int CTRL, int ROWS>
__device__ __forceinline__ double bcast(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, ROWS, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, ROWS, 0xF, false);
  return __hiloint2double(hi, lo);
}
__device__ __forceinline__ float lane_val(float v, int l) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}
__device__ __forceinline__ double lane_val(double v, int l) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), l),
                          __builtin_amdgcn_readlane(__double2loint(v), l));
}

// ---- Products with the lane group's own vector (16-lane groups, FP64). Lane m
// of a 16-lane row holds entry m of its knot's vector; v_fmac_f64 with a
// row_newbcast:m DPP source multiplies every lane's coefficient by that entry
// straight from lane m's register, so the knot's own block-row products need no
// LDS round trip. The terms are accumulated in the same order as the LDS
// form's loops, so the sums are the same bit for bit. Each product is one asm
// statement that starts with the two wait states a DPP read needs after a VALU
// write of its source (x is only read inside it).
#define GATO_NB1(M, C) "v_fmac_f64_dpp %0, %1, %[c" #M "] row_newbcast:" #M " row_mask:0xf bank_mask:0xf\n\t"
#define GATO_C12(c) [c0] "v"(c[0]), [c1] "v"(c[1]), [c2] "v"(c[2]), [c3] "v"(c[3]), [c4] "v"(c[4]), [c5] "v"(c[5]), \
    [c6] "v"(c[6]), [c7] "v"(c[7]), [c8] "v"(c[8]), [c9] "v"(c[9]), [c10] "v"(c[10]), [c11] "v"(c[11])
#define GATO_C14(c) GATO_C12(c), [c12] "v"(c[12]), [c13] "v"(c[13])

// Two 8-lane groups share a row: both groups' products in every lane, of which
// each keeps its own. (Bank masks would keep them apart inside the chain, but a
// masked fmac does not pass the other half's sum on to the next one.)
#define GATO_NB8(M, H, S)                                                                  \
  "v_fmac_f64_dpp %0, " S "%2, %[c" #M "] row_newbcast:" #M " row_mask:0xf bank_mask:0xf\n\t" \
  "v_fmac_f64_dpp %1, " S "%2, %[c" #M "] row_newbcast:" #H " row_mask:0xf bank_mask:0xf\n\t"
#define GATO_DOT8(S)                                                                                            \
  double hi = acc;                                                                                              \
  asm volatile("s_nop 1\n\t" GATO_NB8(0, 8, S) GATO_NB8(1, 9, S) GATO_NB8(2, 10, S)                               \
               GATO_NB8(3, 11, S) GATO_NB8(4, 12, S) GATO_NB8(5, 13, S)                                         \
               : "+v"(acc), "+v"(hi) : "v"(x), [c0] "v"(c[0]), [c1] "v"(c[1]), [c2] "v"(c[2]),                   \
                 [c3] "v"(c[3]), [c4] "v"(c[4]), [c5] "v"(c[5]));                                                \
  acc = (threadIdx.x & 8) ? hi : acc;

// acc += sum_m c[m] x_m, m = 0..NX-1 in order (x_m: x at lane m of the group).
template <int NX>
__device__ __forceinline__ void row_dot1(double &acc, double x, const double *c) {
  static_assert(NX == 6 || NX == 12 || NX == 14, "8-lane groups hold 6 rows, 16-lane groups 12 or 14");
  if constexpr (NX == 6) {
    GATO_DOT8("")
  } else if constexpr (NX == 14) {
    asm volatile("s_nop 1\n\t" GATO_NB1(0, c) GATO_NB1(1, c) GATO_NB1(2, c) GATO_NB1(3, c) GATO_NB1(4, c)
                 GATO_NB1(5, c) GATO_NB1(6, c) GATO_NB1(7, c) GATO_NB1(8, c) GATO_NB1(9, c) GATO_NB1(10, c)
                 GATO_NB1(11, c) GATO_NB1(12, c) GATO_NB1(13, c)
                 : "+v"(acc) : "v"(x), GATO_C14(c));
  } else {
    asm volatile("s_nop 1\n\t" GATO_NB1(0, c) GATO_NB1(1, c) GATO_NB1(2, c) GATO_NB1(3, c) GATO_NB1(4, c)
                 GATO_NB1(5, c) GATO_NB1(6, c) GATO_NB1(7, c) GATO_NB1(8, c) GATO_NB1(9, c) GATO_NB1(10, c)
                 GATO_NB1(11, c)
                 : "+v"(acc) : "v"(x), GATO_C12(c));
  }
}

// acc += sum over the velocity entries m = NX/2..NX-1 only, of coefficients
// c[m - NX/2].
#define GATO_NBV(M, C) "v_fmac_f64_dpp %0, %1, %[c" #C "] row_newbcast:" #M " row_mask:0xf bank_mask:0xf\n\t"
#define GATO_NBV8(C, M, H)                                                             \
  "v_fmac_f64_dpp %0, %2, %[c" #C "] row_newbcast:" #M " row_mask:0xf bank_mask:0xf\n\t" \
  "v_fmac_f64_dpp %1, %2, %[c" #C "] row_newbcast:" #H " row_mask:0xf bank_mask:0xf\n\t"
template <int NX>
__device__ __forceinline__ void row_dot1_vel(double &acc, double x, const double *c) {
  static_assert(NX == 6 || NX == 12 || NX == 14, "8-lane groups hold 6 rows, 16-lane groups 12 or 14");
  if constexpr (NX == 6) {
    double hi = acc;
    asm volatile("s_nop 1\n\t" GATO_NBV8(0, 3, 11) GATO_NBV8(1, 4, 12) GATO_NBV8(2, 5, 13)
                 : "+v"(acc), "+v"(hi) : "v"(x), [c0] "v"(c[0]), [c1] "v"(c[1]), [c2] "v"(c[2]));
    acc = (threadIdx.x & 8) ? hi : acc;
  } else if constexpr (NX == 14) {
    asm volatile("s_nop 1\n\t" GATO_NBV(7, 0) GATO_NBV(8, 1) GATO_NBV(9, 2) GATO_NBV(10, 3) GATO_NBV(11, 4)
                 GATO_NBV(12, 5) GATO_NBV(13, 6)
                 : "+v"(acc) : "v"(x), [c0] "v"(c[0]), [c1] "v"(c[1]), [c2] "v"(c[2]), [c3] "v"(c[3]),
                   [c4] "v"(c[4]), [c5] "v"(c[5]), [c6] "v"(c[6]));
  } else {
    asm volatile("s_nop 1\n\t" GATO_NBV(6, 0) GATO_NBV(7, 1) GATO_NBV(8, 2) GATO_NBV(9, 3) GATO_NBV(10, 4)
                 GATO_NBV(11, 5)
                 : "+v"(acc) : "v"(x), [c0] "v"(c[0]), [c1] "v"(c[1]), [c2] "v"(c[2]), [c3] "v"(c[3]),
                   [c4] "v"(c[4]), [c5] "v"(c[5]));
  }
}
#undef GATO_NBV
#undef GATO_NBV8

// acc -= sum_m c[m] x_m, m = 0..NX-1 in order (the same roundings as
// acc = fma(-c[m], x_m, acc) term by term).
#define GATO_NBN(M, C) "v_fmac_f64_dpp %0, -%1, %[c" #M "] row_newbcast:" #M " row_mask:0xf bank_mask:0xf\n\t"
template <int NX>
__device__ __forceinline__ void row_dot1_sub(double &acc, double x, const double *c) {
  static_assert(NX == 6 || NX == 12 || NX == 14, "8-lane groups hold 6 rows, 16-lane groups 12 or 14");
  if constexpr (NX == 6) {
    GATO_DOT8("-")
  } else if constexpr (NX == 14) {
    asm volatile("s_nop 1\n\t" GATO_NBN(0, c) GATO_NBN(1, c) GATO_NBN(2, c) GATO_NBN(3, c) GATO_NBN(4, c)
                 GATO_NBN(5, c) GATO_NBN(6, c) GATO_NBN(7, c) GATO_NBN(8, c) GATO_NBN(9, c) GATO_NBN(10, c)
                 GATO_NBN(11, c) GATO_NBN(12, c) GATO_NBN(13, c)
                 : "+v"(acc) : "v"(x), GATO_C14(c));
  } else {
    asm volatile("s_nop 1\n\t" GATO_NBN(0, c) GATO_NBN(1, c) GATO_NBN(2, c) GATO_NBN(3, c) GATO_NBN(4, c)
                 GATO_NBN(5, c) GATO_NBN(6, c) GATO_NBN(7, c) GATO_NBN(8, c) GATO_NBN(9, c) GATO_NBN(10, c)
                 GATO_NBN(11, c)
                 : "+v"(acc) : "v"(x), GATO_C12(c));
  }
}
#undef GATO_NBN
#undef GATO_DOT8
#undef GATO_NB8

// acc += sum_m c[m] x_m with FP32 coefficients converted inside the statement (two
// temporaries), m = 0..NX-1 in order; the same roundings as the loop
// acc = fma(c[m], x_m, acc) over the converted c[m].
#define GATO_NBF(M, T) "v_cvt_f64_f32 %[" #T "], %[c" #M "]\n\t"                                \
  "v_fmac_f64_dpp %0, %[x], %[" #T "] row_newbcast:" #M " row_mask:0xf bank_mask:0xf\n\t"
template <int NX>
__device__ __forceinline__ void row_dot1_f(double &acc, double x, const float *c) {
  static_assert(NX == 12 || NX == 14, "16-lane groups hold 12 or 14 rows");
  double ta, tb;
  if constexpr (NX == 14) {
    asm volatile("s_nop 1\n\t" GATO_NBF(0, ta) GATO_NBF(1, tb) GATO_NBF(2, ta) GATO_NBF(3, tb) GATO_NBF(4, ta)
                 GATO_NBF(5, tb) GATO_NBF(6, ta) GATO_NBF(7, tb) GATO_NBF(8, ta) GATO_NBF(9, tb) GATO_NBF(10, ta)
                 GATO_NBF(11, tb) GATO_NBF(12, ta) GATO_NBF(13, tb)
                 : "+v"(acc), [ta] "=&v"(ta), [tb] "=&v"(tb) : [x] "v"(x), GATO_C14(c));
  } else {
    asm volatile("s_nop 1\n\t" GATO_NBF(0, ta) GATO_NBF(1, tb) GATO_NBF(2, ta) GATO_NBF(3, tb) GATO_NBF(4, ta)
                 GATO_NBF(5, tb) GATO_NBF(6, ta) GATO_NBF(7, tb) GATO_NBF(8, ta) GATO_NBF(9, tb) GATO_NBF(10, ta)
                 GATO_NBF(11, tb)
                 : "+v"(acc), [ta] "=&v"(ta), [tb] "=&v"(tb) : [x] "v"(x), GATO_C12(c));
  }
}
// The same over the velocity entries m = NX/2..NX-1 only.
template <int NX>
__device__ __forceinline__ void row_dot1_vel_f(double &acc, double x, const float *c) {
  static_assert(NX == 12 || NX == 14, "16-lane groups hold 12 or 14 rows");
  double ta, tb;
  if constexpr (NX == 14) {
    asm volatile("s_nop 1\n\t" GATO_NBF(7, ta) GATO_NBF(8, tb) GATO_NBF(9, ta) GATO_NBF(10, tb)
                 GATO_NBF(11, ta) GATO_NBF(12, tb) GATO_NBF(13, ta)
                 : "+v"(acc), [ta] "=&v"(ta), [tb] "=&v"(tb)
                 : [x] "v"(x), [c7] "v"(c[7]), [c8] "v"(c[8]), [c9] "v"(c[9]), [c10] "v"(c[10]), [c11] "v"(c[11]),
                   [c12] "v"(c[12]), [c13] "v"(c[13]));
  } else {
    asm volatile("s_nop 1\n\t" GATO_NBF(6, ta) GATO_NBF(7, tb) GATO_NBF(8, ta) GATO_NBF(9, tb)
                 GATO_NBF(10, ta) GATO_NBF(11, tb)
                 : "+v"(acc), [ta] "=&v"(ta), [tb] "=&v"(tb)
                 : [x] "v"(x), [c6] "v"(c[6]), [c7] "v"(c[7]), [c8] "v"(c[8]), [c9] "v"(c[9]), [c10] "v"(c[10]),
                   [c11] "v"(c[11]));
  }
}
#undef GATO_NBF

#undef GATO_NB1
#undef GATO_C12
#undef GATO_C14

// t[c] += s_c * mul for every column c of the group (s_c: s at lane c of the
// row), one term of the row-by-matrix products that form the Schur diagonal
// block: lane c holds row c of the matrix, so its entries need no LDS copy.
#define GATO_RB(C) "v_fmac_f64_dpp %" #C ", %[s], %[m] row_newbcast:" #C " row_mask:0xf bank_mask:0xf\n\t"
template <int NX>
__device__ __forceinline__ void col_fma(double *t, double s, double mul) {
  static_assert(NX == 12 || NX == 14, "16-lane groups hold 12 or 14 rows");
  if constexpr (NX == 14) {
    asm volatile("s_nop 1\n\t" GATO_RB(0) GATO_RB(1) GATO_RB(2) GATO_RB(3) GATO_RB(4) GATO_RB(5) GATO_RB(6)
                 GATO_RB(7) GATO_RB(8) GATO_RB(9) GATO_RB(10) GATO_RB(11) GATO_RB(12) GATO_RB(13)
                 : "+v"(t[0]), "+v"(t[1]), "+v"(t[2]), "+v"(t[3]), "+v"(t[4]), "+v"(t[5]), "+v"(t[6]),
                   "+v"(t[7]), "+v"(t[8]), "+v"(t[9]), "+v"(t[10]), "+v"(t[11]), "+v"(t[12]), "+v"(t[13])
                 : [s] "v"(s), [m] "v"(mul));
  } else {
    asm volatile("s_nop 1\n\t" GATO_RB(0) GATO_RB(1) GATO_RB(2) GATO_RB(3) GATO_RB(4) GATO_RB(5) GATO_RB(6)
                 GATO_RB(7) GATO_RB(8) GATO_RB(9) GATO_RB(10) GATO_RB(11)
                 : "+v"(t[0]), "+v"(t[1]), "+v"(t[2]), "+v"(t[3]), "+v"(t[4]), "+v"(t[5]), "+v"(t[6]),
                   "+v"(t[7]), "+v"(t[8]), "+v"(t[9]), "+v"(t[10]), "+v"(t[11])
                 : [s] "v"(s), [m] "v"(mul));
  }
}
#undef GATO_RB

// One Gauss-Jordan pivot of a lane group (16-lane groups, FP64; lane r holds
// row r): every lane takes the pivot row from lane PV's registers by row
// broadcasts fused into its update, row_c += pivot_c * nf (nf = -f off the
// pivot lane, 0 on it), so no row travels through LDS. The terms and their
// rounding are those of the LDS form.
#define GATO_GJ(C) "v_fmac_f64_dpp %" #C ", %" #C ", %[nf] row_newbcast:%[pv] row_mask:0xf bank_mask:0xf\n\t"
template <int PV, int NX>
__device__ __forceinline__ void gj_pivot(double *row, int lane) {
  static_assert(NX == 12 || NX == 14, "16-lane groups hold 12 or 14 rows");
  double pp = -0.0;   // -0 + x * 1 is x exactly
  asm volatile("s_nop 1\n\tv_fmac_f64_dpp %0, %1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf"
               : "+v"(pp) : "v"(row[PV]), "v"(1.0), "i"(PV));
  const double pinv = 1.0 / pp;
  const double f = row[PV] * pinv;
  const double nf = (lane == PV) ? 0.0 : -f;
  if constexpr (NX == 14) {
    asm volatile("s_nop 1\n\t" GATO_GJ(0) GATO_GJ(1) GATO_GJ(2) GATO_GJ(3) GATO_GJ(4) GATO_GJ(5) GATO_GJ(6)
                 GATO_GJ(7) GATO_GJ(8) GATO_GJ(9) GATO_GJ(10) GATO_GJ(11) GATO_GJ(12) GATO_GJ(13)
                 : "+v"(row[0]), "+v"(row[1]), "+v"(row[2]), "+v"(row[3]), "+v"(row[4]), "+v"(row[5]),
                   "+v"(row[6]), "+v"(row[7]), "+v"(row[8]), "+v"(row[9]), "+v"(row[10]), "+v"(row[11]),
                   "+v"(row[12]), "+v"(row[13])
                 : [nf] "v"(nf), [pv] "i"(PV));
  } else {
    asm volatile("s_nop 1\n\t" GATO_GJ(0) GATO_GJ(1) GATO_GJ(2) GATO_GJ(3) GATO_GJ(4) GATO_GJ(5) GATO_GJ(6)
                 GATO_GJ(7) GATO_GJ(8) GATO_GJ(9) GATO_GJ(10) GATO_GJ(11)
                 : "+v"(row[0]), "+v"(row[1]), "+v"(row[2]), "+v"(row[3]), "+v"(row[4]), "+v"(row[5]),
                   "+v"(row[6]), "+v"(row[7]), "+v"(row[8]), "+v"(row[9]), "+v"(row[10]), "+v"(row[11])
                 : [nf] "v"(nf), [pv] "i"(PV));
  }
  if (lane == PV) {
#pragma unroll
    for (int c = 0; c < NX; ++c)
      if (c != PV) row[c] = row[c] * pinv;
  }
  row[PV] = (lane == PV) ? pinv : -f;
}
template <int NX, int... PV>
__device__ __forceinline__ void gj_dpp(double *row, int lane, std::integer_sequence<int, PV...>) {
  (gj_pivot<PV, NX>(row, lane), ...);
}
#undef GATO_GJ

// The PCG's reciprocals: the hardware reciprocal and two Newton steps (about an ulp
// from the rounded one), instead of a correctly rounded division, whose longer
// dependent chain sits between the inner products and the vector updates of every
// iteration. The all-FP32 variant with FP64 inner products takes its quotients from
// it (div_pcg).
__device__ __forceinline__ double rcp_pcg(double b) {
  double r = __builtin_amdgcn_rcp(b);
  double e = fma(-b, r, 1.0);
  r = fma(r, e, r);
  e = fma(-b, r, 1.0);
  return fma(r, e, r);
}
__device__ __forceinline__ double div_pcg(double a, double b) { return a * rcp_pcg(b); }
__device__ __forceinline__ float div_pcg(float a, float b) { return a / b; }

// Sum over the wavefront (all 64 lanes must be active).
template <class R>
__device__ __forceinline__ R wave_sum(R v) {
  v += dpp<0xB1>(v);   // quad_perm [1,0,3,2]
  v += dpp<0x4E>(v);   // quad_perm [2,3,0,1]
  v += dpp<0x141>(v);  // row_half_mirror
  v += dpp<0x140>(v);  // row_mirror: every lane holds its row's sum
  // Row 3 ends with (r3 + r2) + (r1 + r0), the rows' sums in a fixed order.
  v += bcast<0x142, 0xA>(v);
  v += bcast<0x143, 0xC>(v);
  return lane_val(v, 63);
}

// Sum over the workgroup of NV values: butterfly inside each wavefront, then a
// fixed-order sum of the per-wavefront partials.
// The partials travel through LDS as double (exact for float values).
template <int NV, class V>
__device__ __forceinline__ void block_sum(double (*red)[3][kBlock / 64], int &buf, V *v) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
#pragma unroll
  for (int i = 0; i < NV; ++i) v[i] = wave_sum(v[i]);
  if ((threadIdx.x & 63) == 0) {
#pragma unroll
    for (int i = 0; i < NV; ++i) red[buf][i][wave] = (double)v[i];
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    V s = 0;
#pragma unroll
    for (int w = 0; w < kBlock / 64; ++w) s += (V)red[buf][i][w];
    v[i] = s;
  }
  buf ^= 1;
}

// ---- PCG with the stair preconditioner in two half-sweeps (FP64).
// With D and O the block diagonal and the block off-diagonal of S~, the
// factored preconditioner of Eq. (6), P = D^-1 - D^-1 O D^-1, gives
//   S~ P = (D + O) (D^-1 - D^-1 O D^-1) = I - (O D^-1)^2,
// so one pass of
//   z = D^-1 w,  y = O z,  v = D^-1 y,  m = P w = z - v,  n = S~ m = w - O v
// forms both products of a pipelined iteration without the rows of D: four
// block-row products fewer than P and S~ one after the other need (six against
// seven), and 28 registers per knot of a lane group free. The rows of O are held
// scaled, Am = -A_{k-1} Q_{k-1}^-1 and Ac = -Q_k^-1 A_k^T, so that one vector
// (z, then v) is published per product. Rows that do not exist are zero and the
// knots beyond the ends are zero rows of the buffers, so the loop has no masks.
// Measured against P and S~ applied one after the other (us per PCG iteration,
// MI355X): 7 DoF N = 32, 256 solves 1.49 -> 0.87; N = 64 3.07 -> 1.29 (two
// knots per lane group: the A rows in FP64 and no spills in the loop); 6 DoF
// N = 8 0.94 -> 0.50; tip tracking 7 DoF N = 32 1.54 -> 1.00. The loop of one
// knot per lane group has 117 VALU instructions (237), 72 of them the products.

// Two sums over the workgroup through the matrix cores: three v_mfma_f64_4x4x4
// (lane = i + 4 block + 16 k for A, j + 4 block + 16 k for B, j + 4 block + 16 i
// for the result) leave, per wavefront, the four blocks' sums of `a` in the even
// columns and of `b` in the odd ones; BlockSums::get adds the 32 partials of each
// after the barrier, in the same order in every lane. Against DPP butterflies and
// a pairwise tree over broadcast reads this takes 9 instead of 54 VALU
// instructions per wavefront off the loop, and 2 LDS reads instead of 8.
__device__ __forceinline__ double block_sums_start(int tid, double a, double b) {
  const double even = (tid & 1) ? 0.0 : 1.0;
  const double d = __builtin_amdgcn_mfma_f64_4x4x4f64(a, even, 0.0, 0, 0, 0);
  return __builtin_amdgcn_mfma_f64_4x4x4f64(b, 1.0 - even, d, 0, 0, 0);
}
// (In the pipelined loop every lane writes: no exec mask splits the block that
// the scheduler fills the sums' latency from.)
__device__ __forceinline__ void block_sums_finish(double *red, int tid, double d) {
  d = __builtin_amdgcn_mfma_f64_4x4x4f64(1.0, d, 0.0, 0, 0, 0);
  const int l = tid & 63;
  red[(l & 0x32) == 0 ? (tid >> 6) * 8 + (l >> 2) * 2 + (l & 1) : 64 + l] = d;
}
__device__ __forceinline__ void block_sums_put(double *red, int tid, double a, double b) {
  const double d = __builtin_amdgcn_mfma_f64_4x4x4f64(1.0, block_sums_start(tid, a, b), 0.0, 0, 0, 0);
  const int l = tid & 63;
  if ((l & 0x32) == 0) red[(tid >> 6) * 8 + (l >> 2) * 2 + (l & 1)] = d;
}
struct BlockSums {
  double x[4];
  __device__ __forceinline__ void read(const double *red, int tid) {
    const double *q = red + 4 * ((tid & 3) + 4 * ((tid & 63) >> 4));
#pragma unroll
    for (int i = 0; i < 4; ++i) x[i] = q[i];
  }
  __device__ __forceinline__ void get(double &a, double &b) const {
    const double da = __builtin_amdgcn_mfma_f64_4x4x4f64(x[0] + x[2], 1.0, 0.0, 0, 0, 0);
    const double db = __builtin_amdgcn_mfma_f64_4x4x4f64(x[1] + x[3], 1.0, 0.0, 0, 0, 0);
    a = __builtin_amdgcn_mfma_f64_4x4x4f64(1.0, da, 0.0, 0, 0, 0);
    b = __builtin_amdgcn_mfma_f64_4x4x4f64(1.0, db, 0.0, 0, 0, 0);
  }
};

// The off-diagonal product at one knot of a lane group: y +- (O x)_k at this
// lane's row, xl and xr being its entries of x_{k-1} and x_{k+1}.
// (xs: x_{k+1} at this lane's row for joint rows, at the row of the same joint's
// angle for velocity rows.)
// From rows in registers:
template <int ND, int K>
struct OffRows {
  static constexpr bool shifted = false;
  const double (&Am)[K][2 * ND];
  const double (&Ac)[K][2 * ND];
  __device__ __forceinline__ void add(int p, double &y, double xl, double xr, double) const {
    row_dot1<2 * ND>(y, xl, Am[p]);
    row_dot1<2 * ND>(y, xr, Ac[p]);
  }
  __device__ __forceinline__ void sub(int p, double &y, double xl, double xr, double) const {
    row_dot1_sub<2 * ND>(y, xl, Am[p]);
    row_dot1_sub<2 * ND>(y, xr, Ac[p]);
  }
};
// With the joint rows of A_k known to be [I, hI] (the Euler step's), their part
// of the column of A_k is one entry: Av, the velocity rows' part, and aj, the
// coefficient of xs. 128 -> 117 vector instructions per iteration at one knot per
// lane group and 234 -> 212 at two, the loops' bound (7 DoF, 256 solves of two SQP
// iterations: N = 32 332 -> 322 us; closed-loop tick at N = 64 1690 -> 1616 us).
// Blocks given by the caller and tip tracking's rewritten A_k have no such rows and
// keep OffRows.
template <int ND, int K>
struct OffEuler {
  static constexpr bool shifted = true;
  const double (&Am)[K][2 * ND];
  const double (&Av)[K][ND];
  const double (&aj)[K];
  __device__ __forceinline__ void add(int p, double &y, double xl, double xr, double xs) const {
    row_dot1<2 * ND>(y, xl, Am[p]);
    add_col(p, y, xr, xs);
  }
  __device__ __forceinline__ void sub(int p, double &y, double xl, double xr, double xs) const {
    double t = 0.0;
    add(p, t, xl, xr, xs);
    y -= t;
  }
  __device__ __forceinline__ void add_col(int p, double &y, double xr, double xs) const {
    y += aj[p] * xs;
    row_dot1_vel<2 * ND>(y, xr, Av[p]);
  }
};
// From the velocity rows of A in LDS (four knots per lane group): the row of
// A_{k-1} is read as 2 ND floats, the column of A_k as ND, and the joint rows'
// [I, hI] costs a lane shift each. FULL (caller-given QP data): A_k as it is,
// from the workspace (`full`).
template <int ND, int K, bool FULL>
struct OffLds {
  const float (*Av)[ND][2 * ND];
  const float *full;
  const double (&qown)[K];   // Q_k^-1 at (lane, lane)
  double qi;                 // Q^-1 at (lane, lane)
  double h;
  int lane, slot, N;
  __device__ __forceinline__ bool valid(int p) const { return slot + p * Shape<ND>::SLOTS < N && lane < 2 * ND; }
  // (A_{k-1} Q_{k-1}^-1 x_{k-1}) and (Q_k^-1 A_k^T x_{k+1}) at this lane's row. The
  // block indexes are clamped where no block is: x is zero there.
  __device__ __forceinline__ double row(int p, double xl) const {
    constexpr int NX = 2 * ND;
    const int km = min(max(slot + p * Shape<ND>::SLOTS - 1, 0), N - 2);
    const double g = xl * qi;
    double t = 0.0;
    const float *ar = FULL ? full + ((size_t)km * NX + min(lane, NX - 1)) * NX
                           : Av[km][lane >= ND && lane < NX ? lane - ND : 0];
    float c[NX];
#pragma unroll
    for (int m = 0; m < NX; ++m) c[m] = ar[m];
    row_dot1_f<NX>(t, g, c);
    if constexpr (FULL) {
      return t;
    } else {
      const double up = dpp<0x100 + ND>(g);   // the entry of lane + ND
      return lane < ND ? fma(h, up, g) : t;
    }
  }
  __device__ __forceinline__ double col(int p, double xr) const {
    constexpr int NX = 2 * ND;
    const int kc = min(slot + p * Shape<ND>::SLOTS, N - 2), l = min(lane, NX - 1);
    float c[NX];
    if constexpr (FULL) {
#pragma unroll
      for (int m = 0; m < NX; ++m) c[m] = full[((size_t)kc * NX + m) * NX + l];
      double t = 0.0;
      row_dot1_f<NX>(t, xr, c);
      return qown[p] * t;
    } else {
#pragma unroll
      for (int m = 0; m < ND; ++m) c[ND + m] = Av[kc][m][l];
      const double dn = dpp<0x110 + ND>(xr);   // the entry of lane - ND
      double t = lane < ND ? xr : h * dn;
      row_dot1_vel_f<NX>(t, xr, c);
      return qown[p] * t;
    }
  }
  __device__ __forceinline__ void add(int p, double &y, double xl, double xr) const {
    const double t = row(p, xl) + col(p, xr);
    y -= valid(p) ? t : 0.0;
  }
  __device__ __forceinline__ void sub(int p, double &y, double xl, double xr) const {
    const double t = row(p, xl) + col(p, xr);
    y += valid(p) ? t : 0.0;
  }
  __device__ __forceinline__ void add_col(int p, double &y, double xr, double) const {
    const double t = col(p, xr);
    y -= valid(p) ? t : 0.0;
  }
};

// One knot's share of the Schur complement (Eq. (5)), lane = row: thr, the row of
// D_k = theta_{k-1}; gam, the entry of gamma~; res = gam - (D_k lambda_k). first:
// knot 0, whose block is Q_0^-1. arow(m): the row of A_{k-1}; put(m, x): takes the row of
// O_{k,k-1}; A, B: the blocks
// (A only read by 8-lane groups). Lanes 0..NX-1 of the group.
template <int ND, class Row, class Put>
__device__ __forceinline__ void schur_knot(int lane, bool first, const Row &arow, const Put &put, const float *A, const float *B,
                                           const double *Qi, const double *Qik, const double *Ri, const float *c0,
                                           const float *e, const float *qk, const float *qm, const float *rm,
                                           double lam, double *thr, double &gam, double &res) {
  constexpr int NX = 2 * ND, NU = ND;
  if (first) {
#pragma unroll
    for (int m = 0; m < NX; ++m) thr[m] = (m == lane) ? Qi[lane] : 0.0;
    gam = (double)c0[lane] + Qi[lane] * (double)qk[lane];
  } else {
    double Ar[NX], Br[NU], ArQ[NX], BrR[NU];
#pragma unroll
    for (int m = 0; m < NX; ++m) {
      Ar[m] = arow(m);
      ArQ[m] = Ar[m] * Qi[m];
      put(m, -ArQ[m]);
    }
#pragma unroll
    for (int m = 0; m < NU; ++m) {
      Br[m] = (double)B[lane * NU + m];
      BrR[m] = Br[m] * Ri[m];
    }
    if constexpr (Shape<ND>::G == 16) {
      // Entry (lane, c): the rows of A_{k-1} and B_{k-1} that lane c holds, read
      // by row broadcasts.
#pragma unroll
      for (int c = 0; c < NX; ++c) thr[c] = (c == lane) ? Qik[lane] : 0.0;
#pragma unroll
      for (int m = 0; m < NX; ++m) col_fma<NX>(thr, Ar[m], ArQ[m]);
#pragma unroll
      for (int m = 0; m < NU; ++m) col_fma<NX>(thr, Br[m], BrR[m]);
    } else {
#pragma unroll
      for (int c = 0; c < NX; ++c) {
        double t = (c == lane) ? Qik[lane] : 0.0;
#pragma unroll
        for (int m = 0; m < NX; ++m) t += ArQ[m] * (double)A[c * NX + m];
#pragma unroll
        for (int m = 0; m < NU; ++m) t += BrR[m] * (double)B[c * NU + m];
        thr[c] = t;
      }
    }
    double z = (double)e[lane] + Qik[lane] * (double)qk[lane];
#pragma unroll
    for (int m = 0; m < NX; ++m) z -= ArQ[m] * (double)qm[m];
#pragma unroll
    for (int m = 0; m < NU; ++m) z -= BrR[m] * (double)rm[m];
    gam = z;
  }
  res = gam;
  row_dot1_sub<NX>(res, lam, thr);
}

// The row of D_k^-1 by Gauss-Jordan elimination inside the lane group (the block
// is SPD, so no pivoting is needed). DPP: pivot rows by row broadcasts, else
// through piv (LDS, one row per lane group).
template <int ND, bool DPP>
__device__ __forceinline__ void invert_knot(int lane, bool first, const double *Qi, double *thr, double *piv,
                                            double *Pd) {
  constexpr int NX = 2 * ND;
  if (first) {
    const double d0 = lane < NX ? 1.0 / Qi[lane] : 0.0;
#pragma unroll
    for (int m = 0; m < NX; ++m) Pd[m] = (m == lane) ? d0 : 0.0;
    return;
  }
  if constexpr (DPP) {
    gj_dpp<NX>(thr, lane, std::make_integer_sequence<int, NX>{});
  } else {
#pragma unroll
    for (int pv = 0; pv < NX; ++pv) {
      if (lane == pv) {
#pragma unroll
        for (int c = 0; c < NX; ++c) piv[c] = thr[c];
      }
      wave_sync();
      double prow[NX];
#pragma unroll
      for (int c = 0; c < NX; ++c) prow[c] = piv[c];
      wave_sync();
      const double pinv = 1.0 / prow[pv];
      if (lane == pv) {
#pragma unroll
        for (int c = 0; c < NX; ++c) thr[c] = (c == pv) ? pinv : thr[c] * pinv;
      } else {
        const double f = thr[pv] * pinv;
#pragma unroll
        for (int c = 0; c < NX; ++c) thr[c] = (c == pv) ? -f : thr[c] - f * prow[c];
      }
    }
  }
#pragma unroll
  for (int c = 0; c < NX; ++c) Pd[c] = lane < NX ? thr[c] : 0.0;
}

// A value that is the same in every lane, in scalar registers.
__device__ __forceinline__ double uniform(double v) {
  return __hiloint2double(__builtin_amdgcn_readfirstlane(__double2hiint(v)),
                          __builtin_amdgcn_readfirstlane(__double2loint(v)));
}

// Where u and w are formed from r itself (tip tracking, pcg_long), gamma goes on
// falling for as long as the tolerance asks for it (the pipelined recurrences stall
// some twenty orders of magnitude below its start). Those loops stop here, where
// the scalars are still inside FP64's range; a tolerance further down is reported
// as not reached.
constexpr double kGammaMin = 1e-280;

// What a solve on one workgroup exchanges with others: nothing.
struct NoExchange {
  static constexpr bool on = false;
  __device__ __forceinline__ void put(const double *) {}
  __device__ __forceinline__ void get(double *, double *) {}
  __device__ __forceinline__ void put_sums(double, double) {}
  __device__ __forceinline__ void wait_sums() {}
  __device__ __forceinline__ void get_sums(double &, double &) {}
};

// Runs the PCG from lam (whose off-diagonal product still has to be taken off
// the residual r = gamma~ - D lam) and updates lam. Am, Ac, Pd: this lane's rows
// of the scaled off-diagonal blocks and of D^-1. Returns the iteration count;
// capped: the tolerance was not reached. Per iteration (u = P r, w = S~ u by
// recurrence):
//   gamma = (r, u), delta = (w, u), m = P w, n = S~ m
//   beta = gamma / gamma_prev, alpha = gamma / (delta - beta gamma / alpha_prev)
//   z = n + beta z, q = m + beta q, s = w + beta s, p = u + beta p
//   lambda += alpha p, r -= alpha s, u -= alpha q, w -= alpha z
// PIPE = false (tip tracking): u and w from r itself and a barrier more for the
// sums. The tip systems are conditioned worse (kappa(P S~) about 2e4): there the
// pipelined recurrences stop converging near a tolerance of 1e-8 (the cap of
// 2000 iterations instead of about 300), for 0.96 against 1.00 us per iteration.
// (The parts of a split tip solve run the pipelined loop all the same, since a barrier
// more would be a round trip more between workgroups. They reach 1e-9 in the usual
// count; at 1e-10 some solves of N >= 100 take three to ten times as many.)
// The loop's time is the latency of its two exchanges through LDS next to the
// two wavefronts' FMAs, so everything that hangs on the sums (scalars, stopping
// test) sits where another product is under way; the test is taken after the
// end: a pass begun after convergence is thrown away. NA: the knots per lane of this
// wavefront that exist (for some of its lane groups); a wavefront without any
// only keeps the barriers and the scalars. A split solve's
// parts exchange, at each product, their first and last knot's entries and their
// partial sums (xch; the neighbours' entries stay in the registers of the lane
// groups next to them).
template <int ND, int K, int NA, bool PIPE, class Off, class X>
__device__ __forceinline__ int pcg_half_sweeps(PcgBufs<ND, K> &pb, int tid, int lane, int slot, const Off &o,
                                               X &xch,
                                               const double (&Pd)[K][2 * ND], const double (&gam)[K], double (&r)[K],
                                               double (&lam)[K], double tol, int max_it, bool &capped) {
  constexpr int NX = 2 * ND, SLOTS = Shape<ND>::SLOTS, G = Shape<ND>::G;
  auto each = [&](auto f) {
#pragma unroll
    for (int p = 0; p < NA; ++p) f(p);
  };
  auto publish = [&](double (*buf)[G], const double *x) {
    each([&](int p) { buf[slot + p * SLOTS + 1][lane] = x[p]; });
    xch.put(x);
  };
  auto dinv = [&](const double *x, double *y) {
    each([&](int p) {
      y[p] = 0.0;
      row_dot1<NX>(y[p], x[p], Pd[p]);
    });
  };
  double xl[K], xr[K], xs[K];   // the neighbours' entries of a published vector
  const int lane_s = lane < ND ? lane : lane - ND;
  auto read = [&](const double (*buf)[G]) {
    each([&](int p) {
      xl[p] = buf[slot + p * SLOTS][lane];
      xr[p] = buf[slot + p * SLOTS + 2][lane];
      xs[p] = Off::shifted && !X::on ? buf[slot + p * SLOTS + 2][lane_s] : 0.0;
    });
    xch.get(xl, xr);
    if constexpr (Off::shifted && X::on) {
      each([&](int p) {
        const double angle = dpp<0x110 + ND>(xr[p]);   // the entry of lane - ND
        xs[p] = lane < ND ? xr[p] : angle;
      });
    }
  };
  auto off = [&](double *y) {   // y = O x
    each([&](int p) {
      y[p] = 0.0;
      o.add(p, y[p], xl[p], xr[p], xs[p]);
    });
  };
  auto off_sub = [&](double *y) {   // y -= O x
    each([&](int p) {
      o.sub(p, y[p], xl[p], xr[p], xs[p]);
    });
  };
  double u[K], w[K], z[K], y[K], v[K];
#pragma unroll
  for (int p = 0; p < K; ++p) u[p] = w[p] = z[p] = y[p] = v[p] = 0.0;
  // r = gamma~ - S~ lambda.
  publish(pb.z, lam);
  __syncthreads();
  read(pb.z);
  off_sub(r);
  // P gamma~ (for the reference norm) and u = P r, then w = S~ u. (A buffer is
  // written again only after a barrier behind its last reads.)
  dinv(gam, z);
  publish(pb.v, z);
  __syncthreads();
  read(pb.v);
  off(y);
  dinv(y, w);
  BlockSums sums;
  double eta = 0.0, unused = 0.0;
  each([&](int p) { eta += gam[p] * (z[p] - w[p]); });
  block_sums_put(pb.red, tid, eta, 0.0);
  dinv(r, v);
  publish(pb.z, v);
  __syncthreads();
  sums.read(pb.red, tid);
  sums.get(eta, unused);
  xch.put_sums(eta, 0.0);
  read(pb.z);
  off(y);
  dinv(y, z);
  each([&](int p) { u[p] = v[p] - z[p]; });
  publish(pb.v, z);
  xch.wait_sums();
  __syncthreads();
  read(pb.v);
  xch.get_sums(eta, unused);
  each([&](int p) { w[p] = r[p]; });
  off_sub(w);
  const double stop = tol * tol * eta;
  double vs[K], vp[K];
#pragma unroll
  for (int p = 0; p < K; ++p) vs[p] = vp[p] = 0.0;
  // rg = 1 / gamma_prev and cga = 1 / (gamma_prev alpha_prev) = d_prev /
  // gamma_prev^2 (d: alpha's divisor) turn beta and alpha into two independent
  // reciprocals. (Squares of gamma, which only the pipelined loop keeps in range; the
  // other one has ra = 1 / alpha_prev, for as many operations behind the sums.)
  double rg = 0.0, cga = 0.0;
  int its = 0;
  if constexpr (!PIPE) {
    static_assert(!X::on, "the parts of a split solve run the pipelined loop");
    const double limit = uniform(stop < kGammaMin ? kGammaMin : stop);
    double ra = 0.0;
    for (;;) {
      double pr = 0.0, pw = 0.0;
      each([&](int p) {
        pr += r[p] * u[p];
        pw += w[p] * u[p];
      });
      block_sums_put(pb.red, tid, pr, pw);
      __syncthreads();
      sums.read(pb.red, tid);
      double gma, dlt;
      sums.get(gma, dlt);
      const double beta = gma * rg;
      const double d = dlt - beta * (gma * ra);
      rg = rcp_pcg(gma);
      const double alpha = gma * rcp_pcg(d);
      ra = d * rg;
      capped = gma > stop;
      if (!__builtin_amdgcn_readfirstlane((int)(gma > limit)) || its >= max_it) break;
      each([&](int p) {
        vs[p] = w[p] + beta * vs[p];
        r[p] -= alpha * vs[p];
      });
      dinv(r, z);
      publish(pb.z, z);
      each([&](int p) {
        vp[p] = u[p] + beta * vp[p];
        lam[p] += alpha * vp[p];
      });
      // (Before the barrier, where the wavefront waits anyway: behind it, with one
      // knot per lane, 1.04 against 1.01 us per iteration.)
      if constexpr (K == 1) __builtin_amdgcn_sched_barrier(0);
      __syncthreads();
      read(pb.z);
      off(y);
      dinv(y, v);
      publish(pb.v, v);
      __syncthreads();
      read(pb.v);
      each([&](int p) {
        u[p] = z[p] - v[p];
        w[p] = r[p];
      });
      off_sub(w);
      ++its;
    }
    return its;
  }
  double vz[K], vq[K];
#pragma unroll
  for (int p = 0; p < K; ++p) vz[p] = vq[p] = 0.0;
  for (;;) {
    double pr = 0.0, pw = 0.0;
    each([&](int p) {
      pr += r[p] * u[p];
      pw += w[p] * u[p];
    });
    const double part = block_sums_start(tid, pr, pw);
    dinv(w, z);
    publish(pb.z, z);
    block_sums_finish(pb.red, tid, part);
    __syncthreads();
    double gma, dlt;
    if constexpr (X::on) {
      // This part's sums leave before the wait for the neighbours' entries.
      sums.read(pb.red, tid);
      sums.get(gma, dlt);
      xch.put_sums(gma, dlt);
      read(pb.z);
      off(y);
    } else {
      read(pb.z);
      __builtin_amdgcn_sched_barrier(0);
      sums.read(pb.red, tid);
      off(y);
      sums.get(gma, dlt);
    }
    dinv(y, v);
    publish(pb.v, v);
    xch.wait_sums();
    __syncthreads();
    read(pb.v);
    __builtin_amdgcn_sched_barrier(0);
    xch.get_sums(gma, dlt);
    const double beta = gma * rg;
    const double d = dlt - gma * gma * cga;
    const double rd = rcp_pcg(d);
    rg = rcp_pcg(gma);
    const double alpha = gma * rd;
    cga = d * (rg * rg);
    each([&](int p) {
      vq[p] = (z[p] - v[p]) + beta * vq[p];
      vs[p] = w[p] + beta * vs[p];
      vp[p] = u[p] + beta * vp[p];
      r[p] -= alpha * vs[p];
      u[p] -= alpha * vq[p];
      y[p] = w[p];
    });
    off_sub(y);   // n
    each([&](int p) {
      vz[p] = y[p] + beta * vz[p];
      w[p] -= alpha * vz[p];
    });
    capped = gma > stop;
    if (!__builtin_amdgcn_readfirstlane((int)capped) || its >= max_it) break;
    each([&](int p) { lam[p] += alpha * vp[p]; });
    ++its;
  }
  return its;
}

// The same for four knots per lane group, whose registers hold D^-1 and the
// vectors but not the rows of O (OffLds): one knot at a time between barriers, so
// that only one knot's entries of A are in registers (the loop's scalars in scalar
// registers), and the arrangement with u and w from r (two vectors fewer, one
// barrier more). na: knots per lane of this wavefront that exist. Bound by the conversions and FMAs of 680 VALU
// instructions per wavefront and iteration. 6 DoF N = 128, 512 solves: 17.4 us per
// iteration with all rows read back through L2 (and D^-1 rows in FP32, 5-8% more
// iterations), 3.3 us; the call 15.1 -> 3.0 ms.
template <int ND, int K, class Off>
__device__ __forceinline__ int pcg_long(PcgBufs<ND, K> &pb, int tid, int lane, int slot, int na, const Off &o,
                                        const double (&Pd)[K][2 * ND], const double (&gam)[K], double (&r)[K],
                                        double (&lam)[K], double tol, int max_it, bool &capped) {
  constexpr int NX = 2 * ND, SLOTS = Shape<ND>::SLOTS;
  auto each = [&](auto f) {
#pragma unroll
    for (int p = 0; p < K; ++p)
      if (p < na) f(p, slot + p * SLOTS + 1);
  };
  auto dinv = [&](int p, double x) {
    double y = 0.0;
    row_dot1<NX>(y, x, Pd[p]);
    return y;
  };
  auto off = [&](int p, const double *const x) {   // (O x) at knot p, x: this lane's entry of the knot's row
    double y = 0.0;
    o.add(p, y, x[-Shape<ND>::G], x[Shape<ND>::G]);
    return y;
  };
  BlockSums sums;
  double u[K], w[K], unused;
  each([&](int p, int k) { pb.z[k][lane] = lam[p]; });
  each([&](int p, int k) { pb.v[k][lane] = dinv(p, gam[p]); });
  __syncthreads();
  double eta = 0.0;
  each([&](int p, int k) {
    r[p] -= off(p, &pb.z[k][lane]);
    eta += gam[p] * (pb.v[k][lane] - dinv(p, off(p, &pb.v[k][lane])));
  });
  block_sums_put(pb.red, tid, eta, 0.0);
  __syncthreads();
  sums.read(pb.red, tid);
  sums.get(eta, unused);
  const double stop = uniform(tol * tol * eta), limit = stop < kGammaMin ? kGammaMin : stop;
  double vs[K], vp[K];
#pragma unroll
  for (int p = 0; p < K; ++p) u[p] = w[p] = vs[p] = vp[p] = 0.0;
  double rg = 0.0, ra = 0.0, alpha = 0.0, beta = 0.0;
  // (The first pass only forms u = P r and w = S~ u.)
  for (int its = -1;;) {
    each([&](int p, int k) {
      vs[p] = w[p] + beta * vs[p];
      vp[p] = u[p] + beta * vp[p];
      r[p] -= alpha * vs[p];
      lam[p] += alpha * vp[p];
      pb.z[k][lane] = dinv(p, r[p]);
    });
    ++its;
    __syncthreads();
    each([&](int p, int k) {
      const double v = dinv(p, off(p, &pb.z[k][lane]));
      pb.v[k][lane] = v;
      u[p] = pb.z[k][lane] - v;
    });
    __syncthreads();
    double pr = 0.0, pw = 0.0;
    each([&](int p, int k) {
      w[p] = r[p] - off(p, &pb.v[k][lane]);
      pr += r[p] * u[p];
      pw += w[p] * u[p];
    });
    block_sums_put(pb.red, tid, pr, pw);
    __syncthreads();
    sums.read(pb.red, tid);
    double gma, dlt;
    sums.get(gma, dlt);
    const double bt = gma * rg;
    beta = uniform(bt);
    const double d = dlt - bt * (gma * ra);
    const double rgm = rcp_pcg(gma);
    rg = uniform(rgm);
    alpha = uniform(gma * rcp_pcg(d));
    ra = uniform(d * rgm);
    capped = gma > stop;
    if (!__builtin_amdgcn_readfirstlane((int)(gma > limit)) || its >= max_it) return its;
  }
}

// ---- Exchange between the workgroups (parts) of a split solve. An FP64 value
// travels as two 64-bit words, each holding one 32-bit half of the value under
// a 32-bit tag (launch epoch, exchange number). The words are written and
// polled with relaxed agent-scope atomics: each access is single-copy atomic
// and coherent across the XCDs' L2 caches, so a reader that sees the tag sees
// the half stored with it, and no fence (no whole-L2 write-back or
// invalidation) is needed. Exchange e uses slot e mod kXSlots of the writer; a part
// reuses a slot only after completing later exchanges that every reader of the
// slot had to take part in. Every wait is bounded.
constexpr int kXSlot = 104;                   // words: left row [0, 32), right row [32, 64), sums [64, 104)
constexpr int kXSlots = 8;
constexpr int kXSums = (kXSlot - 64) / 2;     // values of one part's sums region
constexpr int kXLam = 1024;                   // words: multipliers of 32 knots x 16 rows
constexpr int kXPart = kXSlots * kXSlot + kXLam;
constexpr int kXParts = 4;
constexpr int kXSpin = 1 << 17;               // polls before a wait gives up (default)
static_assert(kXParts == kSplitParts && kXParts * kXPart == kXWordsPerSolve, "exchange layout");

__device__ __forceinline__ void xput(unsigned long long *w, unsigned tag, double v) {
  const unsigned long long u = (unsigned long long)__double_as_longlong(v);
  const unsigned long long t = (unsigned long long)tag << 32;
  __hip_atomic_store(w, t | (u & 0xffffffffull), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __hip_atomic_store(w + 1, t | (u >> 32), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// The values stored under `tag` at wa and wb (wb may be null: one value);
// the four words are polled together, so a wait costs one round trip. False
// (values 0) when the wait gave up or `dead` (an earlier wait of the
// workgroup gave up) is set.
__device__ __forceinline__ bool xget2(unsigned long long *wa, unsigned long long *wb, unsigned tag, bool dead,
                                      int spin, double &va, double &vb) {
  va = 0.0;
  vb = 0.0;
  if (dead) return false;
  unsigned long long a0 = 0, a1 = 0, b0 = 0, b1 = 0;
  const unsigned long long t = (unsigned long long)tag;
  for (int n = 0;; ++n) {
    a0 = __hip_atomic_load(wa, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    a1 = __hip_atomic_load(wa + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (wb) {
      b0 = __hip_atomic_load(wb, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      b1 = __hip_atomic_load(wb + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    } else {
      b0 = b1 = t << 32;
    }
    if ((a0 >> 32) == t && (a1 >> 32) == t && (b0 >> 32) == t && (b1 >> 32) == t) break;
    if (n + 1 >= spin) return false;
  }
  va = __longlong_as_double((long long)((a1 << 32) | (a0 & 0xffffffffull)));
  vb = __longlong_as_double((long long)((b1 << 32) | (b0 & 0xffffffffull)));
  return true;
}
__device__ __forceinline__ bool xget(unsigned long long *w, unsigned tag, bool dead, int spin, double &v) {
  double unused;
  return xget2(w, nullptr, tag, dead, spin, v, unused);
}

// A copy of uniform, constant data through scalar loads. The phases that run the
// chain's dynamics take their own copy, through a solve index that the compiler
// takes as new there: the constants stay in SGPRs, where references to the
// descriptor kept them in vector registers across the SQP iterations (in scratch
// for the most part) and loaded them per lane. (One knot per lane group, 7 DoF: 56
// bytes of scratch before, none now.) Each part of a phase takes its own copy: held
// over a whole phase they push the PCG's masks out of the SGPRs.
template <class T>
__device__ __forceinline__ T load_uniform(const T *p) {
  static_assert(sizeof(T) % 4 == 0, "whole words");
  typedef const unsigned __attribute__((address_space(4))) *Words;
  const Words w = (Words)(p);
  unsigned v[sizeof(T) / 4];
#pragma unroll
  for (unsigned i = 0; i < sizeof(T) / 4; ++i) v[i] = w[i];
  T t;
  __builtin_memcpy(&t, v, sizeof(T));
  return t;
}
__device__ __forceinline__ const SolveDesc *fresh_desc(const KArgs &a, int sid) {
  int s = __builtin_amdgcn_readfirstlane(sid);
  asm volatile("" : "+s"(s));
  return a.desc + s;
}
struct CostWeights {
  float Wq[16], Wn[16], Wr[8];   // (as in SolveDesc)
};
static_assert(offsetof(SolveDesc, Wn) - offsetof(SolveDesc, Wq) == offsetof(CostWeights, Wn) &&
                  offsetof(SolveDesc, Wr) - offsetof(SolveDesc, Wq) == offsetof(CostWeights, Wr),
              "the descriptor's weights are copied as one block");
__device__ __forceinline__ CostWeights load_weights(const SolveDesc *d) {
  return load_uniform(reinterpret_cast<const CostWeights *>(d->Wq));
}

// ---- Phase 1 at the knots of the LDS rows row0 .. row0 + nq - 1: defects, merit
// terms (rows from mp_from), A_k's and B_k's columns (stored by put_a, put_b; lane =
// column), and the cos and sin of ntrig rows' joint angles in the rows of dX, which is
// free until the step recovery.
// The time is the chain of one knot's recursions, a wavefront's instructions one
// after the other. So the sines and cosines are formed by a thread per angle, the
// forward dynamics by a thread per knot instead of by one lane per lane group (one or
// two wavefronts for all knots; up to four passes of the lane groups before), its two
// independent halves, inertia and bias, in different wavefronts. 7 DoF N = 32 12.4 ->
// 8.9 us, N = 64 24 -> 18, 32 knots of a split solve's part 11.7 -> 8.8; 6 DoF N = 128
// 44 -> 26, N = 8 10 -> 7.
template <int ND, class SM, class PutA, class PutB>
__device__ __forceinline__ void lq_knots(SM &sm, const KArgs &a, int sid, int tid, int lane, int slot, int nthr,
                                         int row0, int nq, int ntrig, int mp_from, float h,
                                         int &bad_flag, PutA put_a, PutB put_b) {
  constexpr int NX = 2 * ND, NU = ND, SLOTS = Shape<ND>::SLOTS;
  for (int t = tid; t < ntrig * 8; t += nthr) {
    const int k = row0 + t / 8, j = t % 8;
    if (j < ND) sin_cos(sm.X[k][j], &sm.dX[k][ND + j], &sm.dX[k][j]);
  }
  __syncthreads();
  const int half = (nq + 63) & ~63;   // threads of each half: whole wavefronts
  {
    const int t = tid < half ? tid : tid - half, k = row0 + t;
    const bool mine = t < nq;
    const Chain ch = load_uniform(&fresh_desc(a, sid)->chain);
    float L[ND][ND] = {};   // (defined in every lane: not carried from one iteration to the next)
    bool ok = true;
    if (tid < half) {
      if (mine) {
        float cq[ND], sq[ND];
#pragma unroll
        for (int i = 0; i < ND; ++i) {
          cq[i] = sm.dX[k][i];
          sq[i] = sm.dX[k][ND + i];
        }
        ok = fd_inertia<ND>(ch, cq, sq, L);
#pragma unroll
        for (int i = 0; i < ND; ++i)
#pragma unroll
          for (int j = 0; j <= i; ++j) sm.Lf[k][i * (i + 1) / 2 + j] = L[i][j];
      }
    } else if (tid < 2 * half && mine) {
      float q[ND], qd[ND], cq[ND], sq[ND], b[ND];
#pragma unroll
      for (int i = 0; i < ND; ++i) {
        q[i] = sm.X[k][i];
        qd[i] = sm.X[k][ND + i];
        cq[i] = sm.dX[k][i];
        sq[i] = sm.dX[k][ND + i];
      }
      fd_bias<ND>(ch, q, cq, sq, qd, b);
#pragma unroll
      for (int i = 0; i < ND; ++i) sm.qdd[k][i] = b[i];
    }
    __syncthreads();
    if (tid < half && mine) {
      const CostWeights cw = load_weights(fresh_desc(a, sid));
      float q[ND], qd[ND], u[ND], b[ND], qdd[ND];
#pragma unroll
      for (int i = 0; i < ND; ++i) {
        q[i] = sm.X[k][i];
        qd[i] = sm.X[k][ND + i];
        u[i] = sm.U[k][i];
        b[i] = sm.qdd[k][i];
      }
      fd_solve<ND>(L, u, b, qdd);
#pragma unroll
      for (int i = 0; i < ND; ++i) sm.qdd[k][i] = qdd[i];
      float viol = 0.f, cost = 0.f;
#pragma unroll
      for (int i = 0; i < ND; ++i) {
        const float e0 = (q[i] + h * qd[i]) - sm.X[k + 1][i];
        const float e1 = (qd[i] + h * qdd[i]) - sm.X[k + 1][ND + i];
        sm.e[k][i] = e0;
        sm.e[k][ND + i] = e1;
        viol += fabsf(e0) + fabsf(e1);
      }
#pragma unroll
      for (int i = 0; i < NX; ++i) {
        const float d = sm.X[k][i] - sm.xg[i];
        cost += 0.5f * cw.Wq[i] * d * d;
      }
#pragma unroll
      for (int i = 0; i < NU; ++i) cost += 0.5f * cw.Wr[i] * u[i] * u[i];
      if (k >= mp_from) sm.mp0[k] = (double)cost + (double)a.mu * (double)viol;
      if (!ok || !isfinite(viol) || !isfinite(cost)) bad_flag = 1;
    }
    __syncthreads();
  }
  const Chain ch = load_uniform(&fresh_desc(a, sid)->chain);
  for (int t = slot; t < nq; t += SLOTS) {
    const int k = row0 + t;
    if (lane < NX) {
      float q[ND], qd[ND], cq[ND], sq[ND], qdd[ND], col[ND];
#pragma unroll
      for (int i = 0; i < ND; ++i) {
        q[i] = sm.X[k][i];
        qd[i] = sm.X[k][ND + i];
        cq[i] = sm.dX[k][i];
        sq[i] = sm.dX[k][ND + i];
        qdd[i] = sm.qdd[k][i];
      }
      id_tangent<ND>(ch, q, cq, sq, qd, qdd, lane, col);
      float L[ND][ND];
#pragma unroll
      for (int i = 0; i < ND; ++i)
#pragma unroll
        for (int j = 0; j < ND; ++j) L[i][j] = (j <= i) ? sm.Lf[k][i * (i + 1) / 2 + j] : 0.f;
      chol_solve<ND>(L, col);
      put_a(k, col);
      if (lane < ND) {
        float mi[ND];
#pragma unroll
        for (int i = 0; i < ND; ++i) mi[i] = (i == lane) ? 1.f : 0.f;
        chol_solve<ND>(L, mi);
        put_b(k, mi);
      }
    }
  }
}

// ---- Phase 6: the merit terms mp[i][k] of the trial knots (step candidate i, rows
// row0 .. row0 + nst - 1), a thread each. Where two threads per trial knot exist
// (HALVES: bias has space for kBlock / 2 of them), its dynamics' two halves run in
// different wavefronts; otherwise a thread's one after the other, by the same
// instructions, so that a solve's bits do not depend on the size of its workgroup.
// 6 DoF N = 16 6.4 -> 5.0 us, 7 DoF N = 32 8.9 -> 7.4. Returns a number below n_alpha
// in that many threads of wavefronts that are done early (for the terminal terms).
template <int ND, bool TS, bool HALVES, class SM>
__device__ __forceinline__ int ls_trials(SM &sm, const KArgs &a, int sid, const float *We,
                                         const float (*pr)[4], float *bias, int tid, int nthr, int n_alpha, int row0,
                                         int nst, float h) {
  const int ntask = n_alpha * nst;
  const Chain ch = load_uniform(&fresh_desc(a, sid)->chain);
  const int half = (ntask + 63) & ~63;
  const bool halves = HALVES && 2 * half <= nthr;
  const bool second = halves && tid >= half;
  const int step = halves ? half : nthr;
  for (int t0 = 0; t0 < ntask; t0 += step) {
    const int t = t0 + (second ? tid - half : tid);
    const int i = t / nst, k = row0 + (t - i * nst);
    const bool mine = t < ntask;
    float q[ND] = {}, qd[ND] = {}, u[ND] = {}, L[ND][ND] = {}, b[ND] = {}, al = 0.f;
    if (mine) {
      al = sm.alpha[i];
      float cq[ND], sq[ND];
#pragma unroll
      for (int j = 0; j < ND; ++j) {
        q[j] = sm.X[k][j] + al * sm.dX[k][j];
        qd[j] = sm.X[k][ND + j] + al * sm.dX[k][ND + j];
        u[j] = sm.U[k][j] + al * sm.dU[k][j];
      }
#pragma unroll
      for (int j = 0; j < ND; ++j) sin_cos(q[j], &sq[j], &cq[j]);
      if (!second) fd_inertia<ND>(ch, cq, sq, L);
      if (!halves || second) fd_bias<ND>(ch, q, cq, sq, qd, b);
    }
    if constexpr (HALVES) {
      if (halves) {
        if (mine && second) {
#pragma unroll
          for (int j = 0; j < ND; ++j) bias[t * ND + j] = b[j];
        }
        __syncthreads();
        if (mine && !second) {
#pragma unroll
          for (int j = 0; j < ND; ++j) b[j] = bias[t * ND + j];
        }
      }
    }
    if (mine && !second) {
      float qdd[ND];
      fd_solve<ND>(L, u, b, qdd);
      const CostWeights cw = load_weights(fresh_desc(a, sid));
      float viol = 0.f, cost = 0.f;
#pragma unroll
      for (int j = 0; j < ND; ++j) {
        const float x0 = sm.X[k + 1][j] + al * sm.dX[k + 1][j], x1 = sm.X[k + 1][ND + j] + al * sm.dX[k + 1][ND + j];
        viol += fabsf((q[j] + h * qd[j]) - x0) + fabsf((qd[j] + h * qdd[j]) - x1);
        const float d0 = q[j] - sm.xg[j], d1 = qd[j] - sm.xg[ND + j];
        cost += 0.5f * cw.Wq[j] * d0 * d0 + 0.5f * cw.Wq[ND + j] * d1 * d1 + 0.5f * cw.Wr[j] * u[j] * u[j];
      }
      if constexpr (TS) {
        float pt[3];
        tip_position<ND>(ch, q, pt);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          const float d = pt[c] - pr[k][c];
          cost += 0.5f * We[c] * d * d;
        }
      }
      sm.mp[i][k] = (double)cost + (double)a.mu * (double)viol;
    }
  }
  const int i = halves ? tid - half : nthr - 1 - tid;
  return i >= 0 ? i : n_alpha;
}

// ---- Task-space variant: the tip term of one knot, by the knot's lane group.
// Tip position and Jacobian (lane j: one dual-number pass seeded on q_j), the
// residual p(q) - pref and its cost (lane 0), then H = diag(Q_q + rho) +
// J^T W J, its Cholesky factor L (column by column, lane i holding row i,
// pivots broadcast through tq) and L^-1 (lane j forming column j by forward
// substitution). cs: cos and sin of the knot's angles; Jt, pe, mt, tq, Lc, Li: its LDS rows.
template <int ND>
__device__ __forceinline__ void tip_factor(const Chain &ch, const float *cs, const float *pr, const float *We,
                                           const double *Qd, double rho, int lane, float (*Jt)[8], float *pe,
                                           double *mt, double *tq, double *Lc, double *Li, int &bad_flag) {
  if (lane < ND) {
    dual<float> cv[ND], sv[ND], pt[3];
#pragma unroll
    for (int i = 0; i < ND; ++i) {
      cv[i] = dual<float>{cs[i], i == lane ? -cs[ND + i] : 0.f};
      sv[i] = dual<float>{cs[ND + i], i == lane ? cs[i] : 0.f};
    }
    tip_position<ND>(ch, cv, sv, pt);
#pragma unroll
    for (int c = 0; c < 3; ++c) Jt[c][lane] = pt[c].d;
    if (lane == 0) {
      double tc = 0.0;
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const float d = pt[c].v - pr[c];
        pe[c] = d;
        tc += 0.5 * (double)We[c] * (double)d * (double)d;
      }
      *mt = tc;
      if (!isfinite(tc)) bad_flag = 1;
    }
  }
  wave_sync();
  double hr[ND], lr[ND];
#pragma unroll
  for (int j = 0; j < ND; ++j) {
    double t = (j == lane) ? Qd[j] + rho : 0.0;
    if (lane < ND) {
#pragma unroll
      for (int c = 0; c < 3; ++c) t += (double)We[c] * (double)Jt[c][lane] * (double)Jt[c][j];
    }
    hr[j] = t;
    lr[j] = 0.0;
  }
#pragma unroll
  for (int c = 0; c < ND; ++c) {
    if (lane == c) tq[0] = hr[c];
    wave_sync();
    const double piv = tq[0];
    wave_sync();
    if (lane == 0 && !(piv > 0.0)) bad_flag = 1;
    const double dinv = 1.0 / sqrt(piv);
    const double l = (lane >= c && lane < ND) ? hr[c] * dinv : 0.0;   // L[lane][c]
    lr[c] = l;
    if (lane < ND) tq[lane] = l;
    wave_sync();
#pragma unroll
    for (int j = c + 1; j < ND; ++j) hr[j] -= l * tq[j];
    wave_sync();
  }
  if (lane < ND) {
#pragma unroll
    for (int j = 0; j < ND; ++j)
      if (j <= lane) Lc[tri(lane, j)] = lr[j];
  }
  wave_sync();
  if (lane < ND) {
    // Column `lane` of L^-1: rows lane..ND-1 of the solution of L x = e_lane.
    double xs[ND];
#pragma unroll
    for (int i = 0; i < ND; ++i) {
      double t = (i == lane) ? 1.0 : 0.0;
#pragma unroll
      for (int m = 0; m < i; ++m)
        if (m >= lane) t -= Lc[tri(i, m)] * xs[m];
      xs[i] = (i >= lane) ? t / Lc[tri(i, i)] : 0.0;
      if (i >= lane) Li[tri(i, lane)] = xs[i];
    }
  }
}

// Rewrites knot k's QP data in y_k = T_k^-1 x_k, lane `lane` owning state row
// `lane`: row `lane` of A_k -> T_{k+1}^-1 A_k T_k and e_k -> T_{k+1}^-1 e_k
// (when the knot has a successor, `succ`; L1 = L_{k+1}), q_k (with the tip
// term J^T W (p - pref) added) -> T_k^T q_k, and c_0 -> T_0^-1 c_0 (at the
// first knot, `first`). The joint rows of A_k are [I, hI] by construction of
// the Euler step. Lk, Lik: L_k and L_k^-1; tq: the knot's LDS exchange row.
// (Every pointer is valid; the flags say which rows are rewritten, so that
// the LDS accesses keep their address space.)
template <int ND>
__device__ __forceinline__ void tip_rewrite(int lane, bool succ, bool first, float h, const double *Lk,
                                            const double *Lik, const double *L1, float *Ar, float *e, float *qg,
                                            float *c0, const float (*Jt)[8], const float *pe, const float *We,
                                            double *tq) {
  constexpr int NX = 2 * ND;
  if (succ && lane < NX) {
    if (lane < ND) {
      // Row `lane` of [L_{k+1}^T L_k^-T, h L_{k+1}^T].
#pragma unroll
      for (int c = 0; c < ND; ++c) {
        double t = 0.0;
#pragma unroll
        for (int m = 0; m <= c; ++m)
          if (m >= lane) t += L1[tri(m, lane)] * Lik[tri(c, m)];
        Ar[c] = (float)t;
        Ar[ND + c] = c >= lane ? (float)((double)h * L1[tri(c, lane)]) : 0.f;
      }
    } else {
      // Velocity row: its joint columns times L_k^-T.
      float ar[ND];
#pragma unroll
      for (int m = 0; m < ND; ++m) ar[m] = Ar[m];
#pragma unroll
      for (int c = 0; c < ND; ++c) {
        double t = 0.0;
#pragma unroll
        for (int m = 0; m <= c; ++m) t += (double)ar[m] * Lik[tri(c, m)];
        Ar[c] = (float)t;
      }
    }
  }
  double ev = 0.0, cv = 0.0;
  if (lane < ND) {
    double g = (double)qg[lane];
#pragma unroll
    for (int c = 0; c < 3; ++c) g += (double)Jt[c][lane] * (double)We[c] * (double)pe[c];
    tq[lane] = g;
#pragma unroll
    for (int m = 0; m < ND; ++m) {
      if (m >= lane) {
        if (succ) ev += L1[tri(m, lane)] * (double)e[m];
        if (first) cv += Lk[tri(m, lane)] * (double)c0[m];
      }
    }
  }
  wave_sync();
  if (lane < ND) {
    double qh = 0.0;
#pragma unroll
    for (int m = 0; m < ND; ++m)
      if (m <= lane) qh += Lik[tri(lane, m)] * tq[m];
    qg[lane] = (float)qh;
    if (succ) e[lane] = (float)ev;
    if (first) c0[lane] = (float)cv;
  }
  wave_sync();
}

// The multipliers of a knot between the two sets of variables (joint rows,
// lane `lane` holding row `lane`): lambda^ = T_k^T lambda (to y, forward) and
// lambda = T_k^-T lambda^ (back). tq: the knot's LDS exchange row.
template <int ND>
__device__ __forceinline__ double tip_lambda(int lane, bool forward, const double *Lk, const double *Lik, double *tq,
                                             double lam) {
  if (lane < ND) tq[lane] = lam;
  wave_sync();
  double t = lam;
  if (lane < ND) {
    t = 0.0;
#pragma unroll
    for (int m = 0; m < ND; ++m)
      if (m <= lane) t += (forward ? Lik[tri(lane, m)] : Lk[tri(lane, m)]) * tq[m];
  }
  wave_sync();
  return t;
}

// ---- Split long solves, part-local form. A solve of N > 64 knots (6-7 DoF)
// runs on four workgroups (parts), or on two when four per solve do not fit the
// chip; part j owns knots kf = 32 K j .. kl (at most 32 K, possibly none; K = 1 or
// 2) and runs the layout of K knots per lane group over them, with one halo knot
// on each side in LDS:
//   * LQ of its own knots and of the knot left of them (whose A, B, e, q, r the
//     first own Schur row needs), the defects of its own knots (the knot right
//     of them is the halo state);
//   * Schur rows, diagonal-block inverses and PCG rows of its own knots, held
//     in registers as in a short solve; the entries of the knots next to them and
//     the partial inner products travel through device memory (PartExchange);
//   * after the PCG: the multipliers of the halo knots, then the step of the
//     first own knot (the left part's right halo), so that every part holds
//     the step at its own knots and both halos;
//   * the line search over its own knots, the per-candidate partial merits
//     (and the parts' failure flags) summed over the parts in a fixed order,
//     so every part takes the same step, status and damping.
// Part 0 writes the statistics; every part writes its own knots' trajectory
// and multipliers. The same method as the one-workgroup solve; sums are taken
// per part first, so results differ from it at rounding level.
template <int ND, int K>
struct PartSmem {
  using Sh = Shape<ND>;
  static constexpr int G = Sh::G, NX = Sh::NX, NU = Sh::NU, NL = Sh::NL;
  static constexpr int KS = K * Sh::SLOTS;   // own knots at most
  static constexpr int KH = KS + 2;      // with the halo knots: local index li = k - kf + 1
  float X[KH][G];
  float U[KH][8];
  float dX[KH][G];
  float dU[KH][8];
  float e[KH][G];
  float qg[KH][G];
  float rg[KH][8];
  float qdd[KH][8];
  float Lf[KH][NL];
  PcgBufs<ND, K> pcg;      // rows by local index
  double total[2];         // sums over the parts
  double lam[KS][G];       // multipliers between the PCGs
  double piv[Sh::SLOTS][G];
  double mp0[KH];
  double Qi[G], Qni[G];
  double mp[kMaxAlpha][KH];
  double xmp[kMaxAlpha + 1];        // terminal and initial terms of this part, per candidate (+ current)
  double psum[kMaxAlpha + 1];       // this part's partial merits
  double msum[kXParts][kXSums];     // every part's partial merits and flags
  double merit[kMaxAlpha + 1];
  float alpha[kMaxAlpha];
  float xs[G], xg[G], c0[G];
  int bad[2];
  int xfail, xpad[3];
  float A[KH][NX * NX];
  float B[KH][NX * NU];
};

// LDS of the task-space part-local form, placed after PartSmem: the factors
// L_k, L_k^-1 and tip data of the own knots and both halos (the left halo's
// rewritten A, e and q and the last own knot's rewritten A need them).
template <int ND>
struct PartTsSmem {
  static constexpr int KH = Shape<ND>::SLOTS + 2, NL = Shape<ND>::NL;
  double Lc[KH][NL];
  double Li[KH][NL];
  double tq[KH][8];
  double mt[KH];
  float Jt[KH][3][8];
  float pr[KH][4];
  float pe[KH][4];
};
template <int ND>
constexpr size_t part_ts_offset() {
  return (sizeof(PartSmem<ND, 1>) + 15) & ~(size_t)15;
}
template <int ND, int K, bool TS>
constexpr size_t part_smem_bytes() {
  return TS ? part_ts_offset<ND>() + sizeof(PartTsSmem<ND>) : sizeof(PartSmem<ND, K>);
}

// The larger of the two joint-space part forms.
template <int ND>
constexpr size_t long_part_bytes() {
  return sizeof(PartSmem<ND, 2>) > sizeof(PartSmem<ND, 1>) ? sizeof(PartSmem<ND, 2>) : sizeof(PartSmem<ND, 1>);
}

// The exchange of one part in the PCG (pcg_half_sweeps; 7 DoF N = 128 on four
// workgroups 3.0 -> 1.95 us per iteration, 6 DoF N = 100 on two 9.3 -> 2.35; tip
// tracking N = 128 3.2 -> 2.4; two one-way trips of about 0.35 us between idle
// workgroups, twice that under the polling of 200, are on every iteration's path): the first and the last
// own knot's entries of each published vector to the neighbours, theirs into the
// registers of the lane groups that multiply them, and two sums over the parts.
// Vectors and sums count their exchanges separately (hx, sx).
template <int ND, int K>
struct PartExchange {
  static constexpr bool on = true;
  unsigned long long *xb;
  unsigned epoch;
  int part, nparts, spin, tid, lane, slot, slot_r, p_r;   // last own knot: lane group slot_r, p_r-th of it
  bool has_l, has_r;                                      // a neighbour on the left / the right
  int *xfail;
  double *total;                                          // LDS: the sums over the parts
  unsigned hx, sx;
  static constexpr int kSumsWave = 2;
  __device__ __forceinline__ unsigned tag(unsigned e) const { return ((epoch & 0xffffu) << 16) | (e & 0xffffu); }
  __device__ __forceinline__ unsigned long long *at(int q, unsigned e) const {
    return xb + (size_t)q * kXPart + (size_t)(e % kXSlots) * kXSlot;
  }
  __device__ __forceinline__ void put(const double *x) {
    if (lane < 2 * ND) {
      if (has_l && slot == 0) xput(at(part, hx) + 2 * lane, tag(hx), x[0]);
      if (has_r && slot == slot_r) xput(at(part, hx) + 32 + 2 * lane, tag(hx), p_r == 0 ? x[0] : x[K - 1]);
    }
  }
  __device__ __forceinline__ void get(double *xl, double *xr) {
    const bool hl = has_l && slot == 0 && lane < 2 * ND, hr = has_r && slot == slot_r && lane < 2 * ND;
    if (hl || hr) {
      double v;
      if (!xget(hl ? at(part - 1, hx) + 32 + 2 * lane : at(part + 1, hx) + 2 * lane, tag(hx), *xfail != 0, spin, v))
        *xfail = 1;
      if (hl) xl[0] = v;
      else if (p_r == 0) xr[0] = v;
      else xr[K - 1] = v;
    }
    ++hx;
  }
  // One wavefront, next to neither neighbour, sends and collects the sums (with all
  // eight polling the same words an iteration took 2.33 us instead of 1.95): sent as soon as this
  // part's are known, collected into LDS before the barrier behind the next
  // product, whose halo takes as long.
  __device__ __forceinline__ void put_sums(double a, double b) {
    if (tid >> 6 == kSumsWave && (tid & 63) < 2)
      xput(at(part, sx) + 64 + 2 * (tid & 1), tag(sx), tid & 1 ? b : a);
  }
  __device__ __forceinline__ void wait_sums() {
    if (tid >> 6 == kSumsWave) {
      const int l = tid & 63;
      double v = 0.0;
      if (l < 2 * nparts && !xget(at(l >> 1, sx) + 64 + 2 * (l & 1), tag(sx), *xfail != 0, spin, v)) *xfail = 1;
      double a = lane_val(v, 0) + lane_val(v, 2), b = lane_val(v, 1) + lane_val(v, 3);
      if (nparts == 4) {
        a += lane_val(v, 4) + lane_val(v, 6);
        b += lane_val(v, 5) + lane_val(v, 7);
      }
      if (l < 2) total[l] = l ? b : a;
    }
    ++sx;
  }
  __device__ __forceinline__ void get_sums(double &a, double &b) const {
    a = total[0];
    b = total[1];
  }
};

template <int ND, int K, bool TS>
__device__ __attribute__((always_inline)) inline void sqp_solve_part(const KArgs &a, int sid, int part,
                                                                     char *smem_raw) {
  using Sh = Shape<ND>;
  using Real = double;
  constexpr int NX = Sh::NX, NU = Sh::NU, G = Sh::G, SLOTS = Sh::SLOTS;
  static_assert(G == 16, "the part-local split serves 6-7 DoF");
  using SM = PartSmem<ND, K>;
  static_assert(K == 1 || !TS, "tip tracking splits into four parts");
  SM &sm = *reinterpret_cast<SM *>(smem_raw);
  // Only dereferenced by the task-space form, whose LDS holds it.
  PartTsSmem<ND> &ts = *reinterpret_cast<PartTsSmem<ND> *>(smem_raw + part_ts_offset<ND>());
  const SolveDesc &D = a.desc[sid];
  const int tid = threadIdx.x;
  const int lane0 = tid % G;
  const int slot0 = tid / G;
  const int N = D.N;
  const float h = D.dt;
  const int n_alpha = a.n_alpha;
  constexpr int nparts = K == 1 ? kXParts : kXParts / 2;
  constexpr int KS = K * SLOTS;                              // own knots at most
  const bool writer = part == 0;
  const int kf = part * KS;                                  // own knots kf .. kl
  const int nloc = max(0, min(KS, N - kf));
  const int kl = kf + nloc - 1;
  const bool has_l = part > 0 && nloc > 0;                    // a neighbour on the left / the right
  const bool has_r = nloc > 0 && kl + 1 < N;
  const size_t xoff = (size_t)sid * a.N_max * a.nx_max;
  const size_t uoff = (size_t)sid * (a.N_max - 1) * a.nu_max;
  double *gL = a.lam + xoff;
  const int sh = a.shift;
  // Knot of a local index and back.
  auto kof = [&](int li) { return kf - 1 + li; };

  // ---- Stage the iterate (own knots and both halos) and the solve constants.
  for (int t = tid; t < (nloc + 2) * G; t += kBlock) {
    const int li = t / G, j = t % G, k = kof(li);
    const bool in = k >= 0 && k < N && j < NX && nloc > 0;
    sm.X[li][j] = in ? a.X[xoff + (size_t)min(k + sh, N - 1) * a.nx_max + j] : 0.f;
  }
  for (int t = tid; t < (nloc + 1) * 8; t += kBlock) {
    const int li = t / 8, j = t % 8, k = kof(li);
    const bool in = k >= 0 && k <= N - 2 && j < NU && nloc > 0;
    sm.U[li][j] = in ? a.U[uoff + (size_t)min(k + sh, N - 2) * a.nu_max + j] : 0.f;
  }
  if (tid < G) {
    const bool in = tid < NX;
    sm.xs[tid] = in ? a.xs[(size_t)sid * a.nx_max + tid] : 0.f;
    sm.xg[tid] = (in && tid < ND) ? a.goal[(size_t)sid * a.nu_max + tid] : 0.f;
  }
  if constexpr (TS) {
    // Reference tip positions of the own and halo knots (not shifted).
    for (int t = tid; t < (nloc + 2) * 4; t += kBlock) {
      const int li = t / 4, c = t % 4, k = kof(li);
      const bool in = k >= 0 && k < N && c < 3 && nloc > 0;
      ts.pr[li][c] = in ? a.pref[((size_t)sid * a.N_max + k) * 3 + c] : 0.f;
    }
  }
  if (tid == 0) {
    sm.bad[0] = 0;
    sm.bad[1] = 0;
    sm.xfail = 0;
    float al = 1.f;
    for (int i = 0; i < n_alpha; ++i) {
      sm.alpha[i] = al;
      al = al / a.beta;
    }
  }
  double lam[K];
#pragma unroll
  for (int p = 0; p < K; ++p) {
    const int i = slot0 + p * SLOTS;
    lam[p] = (a.warm && i < nloc && lane0 < NX) ? gL[min(kf + i + sh, N - 1) * a.nx_max + lane0] : 0.0;
  }
  // (In LDS outside the PCG, as in sqp_solve.)
  auto park = [&]() {
#pragma unroll
    for (int p = 0; p < K; ++p) sm.lam[slot0 + p * SLOTS][lane0] = lam[p];
  };
  auto unpark = [&]() {
#pragma unroll
    for (int p = 0; p < K; ++p) lam[p] = sm.lam[slot0 + p * SLOTS][lane0];
  };
  park();
  double rho = a.rho[sid];
  // (Rows without a knot and the partial sums of wavefronts without knots are
  // never written in the PCG.)
  for (int t = tid; t < PcgBufs<ND, K>::KH * G; t += kBlock) (&sm.pcg.z[0][0])[t] = (&sm.pcg.v[0][0])[t] = 0.0;
  if (tid < 64) sm.pcg.red[tid] = 0.0;
  PartExchange<ND, K> xch{a.xch + D.xch_off, a.epoch, part, nparts, a.xspin > 0 ? a.xspin : kXSpin, tid, lane0, slot0,
                          (nloc - 1) % SLOTS, nloc > SLOTS ? 1 : 0, has_l, has_r, &sm.xfail, sm.total, 0u, 0u};
  __syncthreads();

  for (int it = 0; it < a.iters; ++it) {
    int lane = lane0, slot = slot0;
    asm volatile("" : "+v"(lane), "+v"(slot));
    if (!a.warm && it > 0) {
#pragma unroll
      for (int p = 0; p < K; ++p) lam[p] = 0.0;
      park();
    }
    if (tid < G) {
      // (Task-space form: the joint block of the rewritten Q_k is the identity.)
      const bool unit = TS && tid < ND;
      sm.Qi[tid] = tid < NX ? (unit ? 1.0 : 1.0 / (D.Qd[tid] + rho)) : 0.0;
      sm.Qni[tid] = tid < NX ? (unit ? 1.0 : 1.0 / (D.QNd[tid] + rho)) : 0.0;
    }
    int &bad_flag = sm.bad[it & 1];
    unsigned long long *clk = (a.clk && tid == 0 && writer) ? a.clk + ((size_t)sid * a.iters + it) * 8 : nullptr;
    unsigned long long cyc0 = 0;
    if (clk) {
      clk[0] = wall_clock64();
      cyc0 = clock64();
    }
    // ================= 1. LQ at knots kq0..kq1 (the own knots and the one left of them).
    const int kq0 = max(kf - 1, 0), kq1 = min(kl, N - 2);
    const int nq = nloc > 0 ? kq1 - kq0 + 1 : 0;
    const int lt0 = kq0 - kf + 1;   // the first of their rows
    const int nt = nloc > 0 ? (has_r ? nloc + 1 : nloc) - lt0 + 1 : 0;   // the rows from there on
    lq_knots<ND>(sm, a, sid, tid, lane, slot, kBlock, lt0, nq, nt, 1, h, bad_flag, [&](int lq, const float *col) {
      float *Ak = sm.A[lq];
#pragma unroll
      for (int i = 0; i < ND; ++i) {
        Ak[i * NX + lane] = (i == lane ? 1.f : 0.f) + (lane == ND + i ? h : 0.f);
        Ak[(ND + i) * NX + lane] = h * col[i] + (lane == ND + i ? 1.f : 0.f);
      }
    }, [&](int lq, const float *mi) {
      float *Bk = sm.B[lq];
#pragma unroll
      for (int i = 0; i < ND; ++i) {
        Bk[i * NU + lane] = 0.f;
        Bk[(ND + i) * NU + lane] = h * mi[i];
      }
    });
    // Gradients at the knots kq0..kl, the initial residual, the terminal and
    // initial merit terms (owners of knot N - 1 and knot 0).
    const int lq0 = kq0 - kf + 1;
    for (int t = tid; t < (nloc > 0 ? nloc + 1 - lq0 : 0) * G; t += kBlock) {
      const int lg = lq0 + t / G, j = t % G, kk = kof(lg);
      const float *W = (kk < N - 1) ? D.Wq : D.Wn;
      sm.qg[lg][j] = j < NX ? W[j] * (sm.X[lg][j] - sm.xg[j]) : 0.f;
      if (kk < N - 1 && j < 8) sm.rg[lg][j] = j < NU ? D.Wr[j] * sm.U[lg][j] : 0.f;
    }
    if (tid < G) sm.c0[tid] = (tid < NX && kf == 0) ? sm.xs[tid] - sm.X[1][tid] : 0.f;
    if (tid == kBlock - 1) {
      double x0 = 0.0;
      if (nloc > 0 && kl == N - 1) {
        float cost = 0.f;
        for (int i = 0; i < NX; ++i) {
          const float d = sm.X[nloc][i] - sm.xg[i];
          cost += 0.5f * D.Wn[i] * d * d;
        }
        x0 += (double)cost;
      }
      if (kf == 0) {
        float viol = 0.f;
        for (int i = 0; i < NX; ++i) viol += fabsf(sm.xs[i] - sm.X[1][i]);
        x0 += (double)a.mu * (double)viol;
      }
      sm.xmp[n_alpha] = x0;
    }
    if constexpr (TS) {
      // The tip terms and the factors L_k, L_k^-1 of the own knots and both halos.
      for (int t = slot; t < nt; t += SLOTS) {
        const int lg = lt0 + t, kk = kof(lg);
        tip_factor<ND>(D.chain, sm.dX[lg], ts.pr[lg], (kk < N - 1) ? D.We : D.WeN, (kk < N - 1) ? D.Qd : D.QNd, rho,
                       lane, ts.Jt[lg], ts.pe[lg], &ts.mt[lg], ts.tq[lg], ts.Lc[lg], ts.Li[lg], bad_flag);
      }
    }
    __syncthreads();
    if (tid == 0) sm.bad[(it + 1) & 1] = 0;
    unpark();
    if constexpr (TS) {
      // Tip costs of the own knots into the merit terms; the QP data of the
      // own knots and the left halo rewritten in y_k = T_k^-1 x_k; then the
      // own warm-start multipliers (lambda^ = T_k^T lambda).
      const int nc = (nloc > 0) ? min(kl, N - 2) - kf + 1 : 0;   // own knots with a control
      for (int t = tid; t < nc; t += kBlock) sm.mp0[1 + t] += ts.mt[1 + t];
      if (tid == 0 && nloc > 0 && kl == N - 1) sm.xmp[n_alpha] += ts.mt[nloc];
      const int nr = nloc > 0 ? nloc + 1 - lq0 : 0;
      for (int t = slot; t < nr; t += SLOTS) {
        const int lg = lq0 + t, kk = kof(lg);
        const bool succ = kk < N - 1;
        tip_rewrite<ND>(lane, succ, kk == 0, h, ts.Lc[lg], ts.Li[lg], ts.Lc[succ ? lg + 1 : lg], sm.A[lg] + lane * NX,
                        sm.e[lg], sm.qg[lg], sm.c0, ts.Jt[lg], ts.pe[lg], succ ? D.We : D.WeN, ts.tq[lg]);
      }
      __syncthreads();
      if (slot < nloc) lam[0] = tip_lambda<ND>(lane, true, ts.Lc[slot + 1], ts.Li[slot + 1], ts.tq[slot + 1], lam[0]);
    }
    if (clk) clk[1] = wall_clock64();

    // ================= 2. Schur rows and diagonal-block inverses of the own knots.
    // (The whole column of A_k for tip tracking and where the exchange, not the FMAs,
    // sets the pace: 1.95 against 2.01 us per iteration with one knot per lane group;
    // OffEuler's with two, 2.27 against 2.35.)
    constexpr bool kRows = TS || K == 1;
    double Am[K][NX], Ac[kRows ? K : 1][NX], Av[K][ND], aj[K], Pd[K][NX], gam[K], res[K], qown[K];
#pragma unroll
    for (int p = 0; p < K; ++p) {
      const int i = slot + p * SLOTS, li = i + 1, k = kf + i;
      double thr[NX];
      gam[p] = res[p] = qown[p] = 0.0;
#pragma unroll
      for (int m = 0; m < NX; ++m) {
        thr[m] = Am[p][m] = Pd[p][m] = 0.0;
        if constexpr (kRows) Ac[p][m] = 0.0;
      }
      aj[p] = 0.0;
#pragma unroll
      for (int m = 0; m < ND; ++m) Av[p][m] = 0.0;
      if (i < nloc) {
        const double *Qik = (k < N - 1) ? sm.Qi : sm.Qni;
        if (lane < NX) {
          qown[p] = Qik[lane];
          const float *A = sm.A[li - 1];
          auto arow = [&](int m) -> double { return (double)A[lane * NX + m]; };
          auto put = [&](int m, double x) { Am[p][m] = x; };
          schur_knot<ND>(lane, k == 0, arow, put, A, sm.B[li - 1], sm.Qi, Qik, D.Ri, sm.c0, sm.e[li - 1], sm.qg[li],
                         sm.qg[li - 1], sm.rg[li - 1], lam[p], thr, gam[p], res[p]);
          if (k < N - 1) {
            const float *An = sm.A[li];
            if constexpr (kRows) {
#pragma unroll
              for (int m = 0; m < NX; ++m) Ac[p][m] = -qown[p] * (double)An[m * NX + lane];
            } else {
              aj[p] = -qown[p] * (lane < ND ? 1.0 : (double)h);
#pragma unroll
              for (int m = 0; m < ND; ++m) Av[p][m] = -qown[p] * (double)An[(ND + m) * NX + lane];
            }
          }
        }
        invert_knot<ND, !TS>(lane, k == 0, sm.Qi, thr, sm.piv[slot], Pd[p]);
      }
    }
    if (clk) {
      clk[2] = wall_clock64();
      clk[3] = clk[2];
    }
    // ================= 3-4. Preconditioned CG, entries and sums through the exchange.
    const int max_it = a.pcg_max_iter > 0 ? a.pcg_max_iter : N * NX;
    const int slot_w = (__builtin_amdgcn_readfirstlane(tid) >> 6) * (64 / G);   // the wavefront's first lane group
    auto off = [&]() {
      if constexpr (kRows) return OffRows<ND, K>{Am, Ac};
      else return OffEuler<ND, K>{Am, Av, aj};
    }();
    bool capped = false;
    int its;
    if (K > 1 && slot_w + SLOTS < nloc)
      its = pcg_half_sweeps<ND, K, K, true>(sm.pcg, tid, lane, slot, off, xch, Pd, gam, res, lam, a.pcg_tol, max_it,
                                            capped);
    else if (slot_w < nloc)
      its = pcg_half_sweeps<ND, K, 1, true>(sm.pcg, tid, lane, slot, off, xch, Pd, gam, res, lam, a.pcg_tol, max_it,
                                            capped);
    else
      its = pcg_half_sweeps<ND, K, 0, true>(sm.pcg, tid, lane, slot, off, xch, Pd, gam, res, lam, a.pcg_tol, max_it,
                                            capped);
    unsigned status = capped ? GATO_ST_PCG_MAXITER : 0u;
    if (clk) clk[4] = wall_clock64();

    // ================= 5. Step dZ = -G^-1 (g - C^T lambda) at the own knots and the halos.
    // Multipliers of the halo knots first (exchange), then the own steps and the
    // left halo's step (this part holds its LQ data), then the right halo's step
    // from the right part (its first own knot).
    // (z: last read before the last barrier of the PCG's loop.)
    double (*lv)[G] = sm.pcg.z;
#pragma unroll
    for (int p = 0; p < K; ++p) lv[slot + p * SLOTS + 1][lane] = lam[p];
    xch.put(lam);
    {
      double xl[K], xr[K];
      xch.get(xl, xr);
      if (has_l && slot == 0 && lane < NX) lv[0][lane] = xl[0];
      if (has_r && slot == xch.slot_r && lane < NX) lv[nloc + 1][lane] = xch.p_r == 0 ? xr[0] : xr[K - 1];
    }
    __syncthreads();
    auto step_at = [&](int lg, int kk, Real lam_own, Real qk) {   // step of knot kk (local lg), row `lane`
      Real sx = (Real)sm.qg[lg][lane] - lam_own;
      if (kk < N - 1) {
        const float *A = sm.A[lg];
#pragma unroll
        for (int m = 0; m < NX; ++m) sx += (Real)A[m * NX + lane] * lv[lg + 1][m];
      }
      const float dx = (float)(-qk * sx);
      sm.dX[lg][lane] = dx;
      if (!isfinite(dx)) bad_flag = 1;
      if constexpr (TS) {
        if (lane < ND) ts.tq[lg][lane] = (double)(-qk * sx);
      }
      if (lane < NU && kk < N - 1) {
        const float *B = sm.B[lg];
        Real su = (Real)sm.rg[lg][lane];
#pragma unroll
        for (int m = 0; m < NX; ++m) su += (Real)B[m * NU + lane] * lv[lg + 1][m];
        const float du = (float)(-(Real)D.Ri[lane] * su);
        sm.dU[lg][lane] = du;
        if (!isfinite(du)) bad_flag = 1;
      }
    };
#pragma unroll
    for (int p = 0; p < K; ++p) {
      const int i = slot + p * SLOTS;
      if (i < nloc && lane < NX) step_at(i + 1, kf + i, lam[p], qown[p]);
    }
    if (has_l && slot == 0 && lane < NX) step_at(0, kf - 1, lv[0][lane], (Real)sm.Qi[lane]);
    if constexpr (TS) {
      // Back to x: dx_k = T_k dy_k (joint rows L_k^-T dy) at the own knots and
      // the left halo, and lambda = T_k^-T lambda^ at the own knots.
      auto to_x = [&](int lg) {
        wave_sync();
        double t = 0.0;
        if (lane < ND) {
#pragma unroll
          for (int m = 0; m < ND; ++m)
            if (m >= lane) t += ts.Li[lg][tri(m, lane)] * ts.tq[lg][m];
        }
        wave_sync();
        if (lane < ND) {
          const float dx = (float)t;
          sm.dX[lg][lane] = dx;
          if (!isfinite(dx)) bad_flag = 1;
        }
      };
      if (slot < nloc) {
        const int li = slot + 1;
        to_x(li);
        lam[0] = tip_lambda<ND>(lane, false, ts.Lc[li], ts.Li[li], ts.tq[li], lam[0]);
      }
      if (has_l && slot == 0) to_x(0);
    }
    park();
    __syncthreads();
    {
      // The first own knot's step to the left: a part reads its right neighbour's
      // into dX[nloc + 1].
      double first[K], xl[K], xr[K];
#pragma unroll
      for (int p = 0; p < K; ++p) first[p] = (double)sm.dX[1][lane];
      xch.put(first);
      xch.get(xl, xr);
      if (has_r && slot == xch.slot_r && lane < NX) sm.dX[nloc + 1][lane] = (float)(xch.p_r == 0 ? xr[0] : xr[K - 1]);
    }
    __syncthreads();
    if (clk) clk[5] = wall_clock64();

    // ================= 6. Line search over the own knots; partial merits summed over the parts.
    const int nst = (nloc > 0) ? min(kl, N - 2) - kf + 1 : 0;   // own knots with a control
    static_assert(kBlock / 2 * ND <= (K * SLOTS + 2) * NX * NX, "biases of the trial knots");
    if (const int i = ls_trials<ND, TS, K == 1>(sm, a, sid, D.We, ts.pr, &sm.A[0][0], tid, kBlock, n_alpha, 1,
                                                max(nst, 0), h);
        i < n_alpha) {
      const float al = sm.alpha[i];
      double x0 = 0.0;
      if (nloc > 0 && kl == N - 1) {
        float cost = 0.f;
        for (int j = 0; j < NX; ++j) {
          const float d = (sm.X[nloc][j] + al * sm.dX[nloc][j]) - sm.xg[j];
          cost += 0.5f * D.Wn[j] * d * d;
        }
        if constexpr (TS) {
          float q[ND], pt[3];
#pragma unroll
          for (int j = 0; j < ND; ++j) q[j] = sm.X[nloc][j] + al * sm.dX[nloc][j];
          tip_position<ND>(D.chain, q, pt);
#pragma unroll
          for (int c = 0; c < 3; ++c) {
            const float d = pt[c] - ts.pr[nloc][c];
            cost += 0.5f * D.WeN[c] * d * d;
          }
        }
        x0 += (double)cost;
      }
      if (kf == 0) {
        float viol = 0.f;
        for (int j = 0; j < NX; ++j) viol += fabsf(sm.xs[j] - (sm.X[1][j] + al * sm.dX[1][j]));
        x0 += (double)a.mu * (double)viol;
      }
      sm.xmp[i] = x0;
    }
    __syncthreads();
    if (tid <= n_alpha) {
      double sum = 0.0;
      for (int lg = 1; lg <= max(nst, 0); ++lg) sum += (tid == n_alpha) ? sm.mp0[lg] : sm.mp[tid][lg];
      sm.psum[tid] = sum + sm.xmp[tid];
    }
    __syncthreads();
    {
      // Partial merits (n_alpha + 1), this part's non-finite flag and its
      // exchange failure flag to every part; summed in part order.
      const int nv = n_alpha + 3;
      if (tid < nv) {
        const double v = tid <= n_alpha ? sm.psum[tid] : (tid == n_alpha + 1 ? (double)bad_flag : (double)sm.xfail);
        xput(xch.at(part, xch.sx) + 64 + 2 * tid, xch.tag(xch.sx), v);
      }
      const bool dead = sm.xfail != 0;
      if (tid < nv * nparts) {
        const int q = tid / nv, v = tid % nv;
        double x;
        if (!xget(xch.at(q, xch.sx) + 64 + 2 * v, xch.tag(xch.sx), dead, xch.spin, x)) sm.xfail = 1;
        sm.msum[q][v] = x;
      }
      ++xch.sx;
      __syncthreads();
      if (tid <= n_alpha) {
        double m = 0.0;
        for (int q = 0; q < nparts; ++q) m += sm.msum[q][tid];
        sm.merit[tid] = m;
      }
      __syncthreads();
    }
    int best = -1;
    for (int i = 0; i < n_alpha; ++i) {
      const double m = sm.merit[i];
      if (isfinite(m) && (best < 0 || m < sm.merit[best])) best = i;
    }
    bool any_bad = false, any_xfail = sm.xfail != 0;
    for (int q = 0; q < nparts; ++q) {
      any_bad = any_bad || sm.msum[q][n_alpha + 1] != 0.0;
      any_xfail = any_xfail || sm.msum[q][n_alpha + 2] != 0.0;
    }
    const bool bad = any_bad || best < 0;
    if (bad) status |= GATO_ST_NONFINITE;
    else if (!(sm.merit[best] < sm.merit[n_alpha])) status |= GATO_ST_NO_DESCENT;
    if (any_xfail) status |= GATO_ST_EXCHANGE;
    const double rho_used = rho;
    if (a.rho_adapt) rho = (status & (GATO_ST_NONFINITE | GATO_ST_NO_DESCENT)) ? fmin(2.0 * rho, 1e8) : rho / 3.0;
    const float al = bad ? 0.f : sm.alpha[best];
    if (!bad) {
      for (int t = tid; t < (nloc + 2) * G; t += kBlock) {
        const int lg = t / G, j = t % G, kk = kof(lg);
        if (kk < 0 || kk >= N || nloc == 0) continue;
        sm.X[lg][j] += al * sm.dX[lg][j];
        if (kk < N - 1 && lg <= nloc && j < 8) sm.U[lg][j] += al * sm.dU[lg][j];
      }
    }
    if (tid == 0 && a.stats && writer) {
      gato_solve_stats st;
      st.merit0 = (float)sm.merit[n_alpha];
      st.merit = bad ? (float)sm.merit[n_alpha] : (float)sm.merit[best];
      st.alpha = al;
      st.pcg_iters = its;
      st.status = status;
      st.rho = (float)rho_used;
      a.stats[(size_t)sid * a.stats_stride + it] = st;
    }
    __syncthreads();
    if (clk) {
      clk[6] = wall_clock64();
      clk[7] = clock64() - cyc0;
    }
  }

  // ---- Write back the own knots' iterate and multipliers, and the damping.
  if (writer && a.rho_adapt && tid == 0) a.rho[sid] = rho;
  for (int t = tid; t < nloc * G; t += kBlock) {
    const int lg = 1 + t / G, j = t % G, kk = kof(lg);
    if (j < NX) a.X[xoff + (size_t)kk * a.nx_max + j] = sm.X[lg][j];
    if (kk < N - 1 && j < NU) a.U[uoff + (size_t)kk * a.nu_max + j] = sm.U[lg][j];
  }
  unpark();
#pragma unroll
  for (int p = 0; p < K; ++p) {
    const int i = slot0 + p * SLOTS;
    if (i < nloc && lane0 < NX) gL[(kf + i) * a.nx_max + lane0] = lam[p];
  }
}

// KKT (four knots per lane group, FP64): the kernels of caller-given QP data, whose
// products read whole A blocks. They are kernels of their own for their registers:
// in one with the Euler step's products, those ran 8% slower (7 DoF, N = 128).
template <int ND, int KPT, class Real, bool TS = false, bool SPLIT = false, bool KKT = false>
__device__ __attribute__((always_inline)) inline void sqp_solve(const KArgs &a, int sid, int part, char *smem_raw) {
  using Sh = Shape<ND>;
  constexpr int NX = Sh::NX, NU = Sh::NU, G = Sh::G, SLOTS = Sh::SLOTS;
  using BS = BlockStore<ND, KPT, Real, TS>;
  constexpr bool kHalf = half_sweeps<Real, KPT>();
  constexpr bool kLong = long_form<Real, KPT>();
  using SM = Smem<ND, KPT, Real, TS>;
  if constexpr (kLong) __builtin_assume((a.mode == kModeKkt) == KKT);
  SM &sm = *reinterpret_cast<SM *>(smem_raw);
  // Only dereferenced by the task-space variant, whose LDS holds it.
  TsSmem<ND, KPT> &ts = *reinterpret_cast<TsSmem<ND, KPT> *>(smem_raw + ts_offset<ND, KPT, Real>());
  const SolveDesc &D = a.desc[sid];
  const int tid = threadIdx.x;
  const int lane0 = tid % G;
  const int slot0 = tid / G;
  const int N = D.N;
  const float h = D.dt;
  const int n_alpha = a.n_alpha;
  // Split solve (four knots per lane group): four (or two) workgroups run
  // the same SQP iteration, each with its own workspace, and share the PCG:
  // part j owns the knots of p == j (or p == 2 j, 2 j + 1). Only part 0 writes
  // results.
  // (SPLIT: compiled into kernels of their own, so that the one-workgroup
  // kernels carry none of the exchange code.)
  constexpr bool kSplitOk = SPLIT && (KPT == 4) && !TS;
  // a.split = 4: part j owns p = j; a.split = 2 (when four workgroups per solve
  // do not fit the chip): part j owns p = 2 j and 2 j + 1.
  const int nparts = a.split == 2 ? 2 : kXParts;
  const int psh = nparts == 2 ? 1 : 0;
  const bool split = kSplitOk && a.split && a.mode == kModeSqp && D.xch_off >= 0 && part >= 0 && part < nparts;
  // The parts of a long FP64 solve run the part-local form (one or two knots per
  // lane group over the part's own knots); those of the all-FP32 variant the
  // four-knots-per-group form below.
  if constexpr (kSplitOk && sizeof(Real) == 8) {
    if (split && !a.by_block) {
      if (nparts == kXParts) sqp_solve_part<ND, 1, false>(a, sid, part, smem_raw);
      else sqp_solve_part<ND, 2, false>(a, sid, part, smem_raw);
      return;
    }
  }
  const bool writer = !split || part == 0;
  char *ws = a.ws + D.ws_off + (split ? (int64_t)part * D.ws_part : 0);
  const size_t xoff = (size_t)sid * a.N_max * a.nx_max;
  const size_t uoff = (size_t)sid * (a.N_max - 1) * a.nu_max;
  double *gL = a.lam + xoff;  // [N][nx_max]
  const int rid = a.by_block ? (int)blockIdx.x : sid;  // index of xs, goal, stats
  const int sh = a.shift;

  // Block accessors (LDS or the solve's workspace).
  auto Ablk = [&](int k) -> float * {
    if constexpr (BS::kLds) return sm.A[k];
    else return reinterpret_cast<float *>(ws + D.offA) + (size_t)k * NX * NX;
  };
  auto Bblk = [&](int k) -> float * {
    if constexpr (BS::kLds) return sm.B[k];
    else return reinterpret_cast<float *>(ws + D.offB) + (size_t)k * NX * NU;
  };
  auto Dblk = [&](int k) -> float * {
    if constexpr (BS::kLds) return sm.Dinv[k];
    else return reinterpret_cast<float *>(ws + D.offD) + (size_t)k * NX * NX;
  };
  auto Pblk = [&](int k) -> float * {   // explicit preconditioner blocks: kpt == 1 only
    if constexpr (BS::kLds) return sm.Poff[k];
    else return nullptr;
  };
  // Rows of the Schur diagonal blocks, kept in the workspace (read back through
  // L2) when four knots per lane group would not fit them in registers.
  constexpr bool kThGlobal = KPT >= 4;
  auto Tblk = [&](int k) -> Real * { return reinterpret_cast<Real *>(ws + D.offT) + (size_t)k * NX * NX; };

  // (One knot per lane group: the launch's own workgroup size, block_threads().)
  const int nthr = KPT == 1 ? (int)blockDim.x : kBlock;

  // ---- Stage the iterate and the solve constants in LDS.
  // (With a warm-start shift, knot k starts from the previous knot k + shift,
  // the last knot repeated.)
  for (int t = tid; t < N * G; t += nthr) {
    const int k = t / G, j = t % G;
    const int ks = min(k + sh, N - 1);
    sm.X[k][j] = (j < NX && a.mode != kModeKkt) ? a.X[xoff + (size_t)ks * a.nx_max + j] : 0.f;
  }
  for (int t = tid; t < (N - 1) * 8; t += nthr) {
    const int k = t / 8, j = t % 8;
    const int ks = min(k + sh, N - 2);
    sm.U[k][j] = (j < NU && a.mode != kModeKkt) ? a.U[uoff + (size_t)ks * a.nu_max + j] : 0.f;
  }
  if (tid < G) {
    const bool in = tid < NX && a.mode != kModeKkt;
    sm.xs[tid] = in ? a.xs[(size_t)rid * a.nx_max + tid] : 0.f;
    sm.xg[tid] = (in && tid < ND) ? a.goal[(size_t)rid * a.nu_max + tid] : 0.f;
  }
  if constexpr (TS) {
    // Reference tip positions of this request's horizon (not shifted).
    for (int t = tid; t < N * 4; t += nthr) {
      const int k = t / 4, c = t % 4;
      ts.pr[k][c] = c < 3 ? a.pref[((size_t)sid * a.N_max + k) * 3 + c] : 0.f;
    }
  }
  if (tid == 0) {
    sm.bad[0] = 0;
    sm.bad[1] = 0;
    sm.xfail = 0;
    float al = 1.f;
    for (int i = 0; i < n_alpha; ++i) {
      sm.alpha[i] = al;
      al = al / a.beta;
    }
  }

  if constexpr (kHalf && !kLong) {
    // (Knots beyond the horizon and the partial sums of wavefronts without
    // knots, or of those a smaller workgroup has not, are never written in the PCG.)
    for (int t = tid; t < PcgBufs<ND, KPT>::KH * G; t += nthr) (&sm.pcg.z[0][0])[t] = (&sm.pcg.v[0][0])[t] = 0.0;
    if (tid < 64) sm.pcg.red[tid] = 0.0;
  }
  if constexpr (!kHalf && KPT == 1) {
    if (tid < 2 * 3 * (kBlock / 64)) (&sm.red[0][0][0])[tid] = 0.0;
  }
  // Multipliers of the rows this thread owns (warm start across iterations).
  Real lam[KPT];
#pragma unroll
  for (int p = 0; p < KPT; ++p) {
    const int k = slot0 + p * SLOTS;
    lam[p] = (a.warm && a.mode == kModeSqp && k < N && lane0 < NX)
                 ? (Real)gL[min(k + sh, N - 1) * a.nx_max + lane0] : (Real)0;
  }
  // (FP64 variants: in LDS outside the PCG, which needs the registers of their live
  // range through the other phases.)
  auto park = [&]() {
    if constexpr (kHalf) {
#pragma unroll
      for (int p = 0; p < KPT; ++p) sm.lam[slot0 + p * SLOTS][lane0] = lam[p];
    }
  };
  auto unpark = [&]() {
    if constexpr (kHalf) {
#pragma unroll
      for (int p = 0; p < KPT; ++p) lam[p] = sm.lam[slot0 + p * SLOTS][lane0];
    }
  };
  park();
  int redbuf = 0;
  unsigned xe = 0;   // split solve: exchange number (the same sequence in every part)
  // Damping on every Q_k (Sec. IV-C); uniform across the workgroup.
  double rho = a.rho[sid];
  __syncthreads();

  for (int it = 0; it < a.iters; ++it) {
    // Opaque per-iteration copies: keeps the compiler from hoisting the many
    // lane-dependent selects of the phases below out of the iteration loop,
    // where they would stay live across every phase and spill.
    int lane = lane0, slot = slot0;
    asm volatile("" : "+v"(lane), "+v"(slot));
    // Without warm starts every PCG solve starts from zero.
    if (!a.warm && it > 0) {
#pragma unroll
      for (int p = 0; p < KPT; ++p) lam[p] = (Real)0;
      park();
    }
    // Q^-1 and Q_N^-1 for this iteration's rho (first read after phase 1's barrier).
    // (Task-space variant: the joint block of the rewritten Q_k is the identity.)
    if (tid < G) {
      const bool unit = TS && tid < ND;
      sm.Qi[tid] = tid < NX ? (unit ? 1.0 : 1.0 / (D.Qd[tid] + rho)) : 0.0;
      sm.Qni[tid] = tid < NX ? (unit ? 1.0 : 1.0 / (D.QNd[tid] + rho)) : 0.0;
    }
    int &bad_flag = sm.bad[it & 1];
    unsigned long long *clk = (a.clk && tid == 0 && writer) ? a.clk + ((size_t)sid * a.iters + it) * 8 : nullptr;
    unsigned long long cyc0 = 0;
    if (clk) {
      clk[0] = wall_clock64();
      cyc0 = clock64();
    }
    // ================= 1. LQ: dynamics, derivatives, defects, gradients.
    if (a.mode != kModeKkt) {
      lq_knots<ND>(sm, a, sid, tid, lane, slot, nthr, 0, N - 1, N, 0, h, bad_flag, [&](int k, const float *col) {
        if constexpr (kLong) {
#pragma unroll
          for (int i = 0; i < ND; ++i) sm.Av[k][i][lane] = h * col[i] + (lane == ND + i ? 1.f : 0.f);
        }
        if (!kLong || a.mode == kModeLq) {
          float *Ak = Ablk(k);
#pragma unroll
          for (int i = 0; i < ND; ++i) {
            Ak[i * NX + lane] = (i == lane ? 1.f : 0.f) + (lane == ND + i ? h : 0.f);
            Ak[(ND + i) * NX + lane] = h * col[i] + (lane == ND + i ? 1.f : 0.f);
          }
        }
      }, [&](int k, const float *mi) {
        float *Bk = Bblk(k);
#pragma unroll
        for (int i = 0; i < ND; ++i) {
          Bk[i * NU + lane] = 0.f;
          Bk[(ND + i) * NU + lane] = h * mi[i];
        }
      });
      for (int t = tid; t < N * G; t += nthr) {
        const int k = t / G, j = t % G;
        const float *W = (k < N - 1) ? D.Wq : D.Wn;
        sm.qg[k][j] = j < NX ? W[j] * (sm.X[k][j] - sm.xg[j]) : 0.f;
        if (k < N - 1 && j < 8) sm.rg[k][j] = j < NU ? D.Wr[j] * sm.U[k][j] : 0.f;
      }
      if (tid < G) sm.c0[tid] = tid < NX ? sm.xs[tid] - sm.X[0][tid] : 0.f;
      if (tid == nthr - 1) {
        float cost = 0.f, viol = 0.f;
        for (int i = 0; i < NX; ++i) {
          const float d = sm.X[N - 1][i] - sm.xg[i];
          cost += 0.5f * D.Wn[i] * d * d;
          viol += fabsf(sm.xs[i] - sm.X[0][i]);
        }
        sm.mp0[N - 1] = (double)cost + (double)a.mu * (double)viol;
      }
      if constexpr (TS) {
        // The tip terms and the factors L_k, L_k^-1 of every knot.
        for (int k = slot; k < N; k += SLOTS)
          tip_factor<ND>(D.chain, sm.dX[k], ts.pr[k], (k < N - 1) ? D.We : D.WeN, (k < N - 1) ? D.Qd : D.QNd, rho, lane,
                         ts.Jt[k], ts.pe[k], &ts.mt[k], ts.tq[k], ts.Lc[k], ts.Li[k], bad_flag);
      }
      if (a.mode == kModeLq) {
        __syncthreads();
        const size_t ao = (size_t)sid * (a.N_max - 1) * a.nx_max * a.nx_max;
        const size_t bo = (size_t)sid * (a.N_max - 1) * a.nx_max * a.nu_max;
        const size_t eo = (size_t)sid * (a.N_max - 1) * a.nx_max;
        for (int t = tid; t < (N - 1) * NX * NX; t += nthr) {
          const int k = t / (NX * NX), r = (t / NX) % NX, c = t % NX;
          a.outA[ao + ((size_t)k * a.nx_max + r) * a.nx_max + c] = Ablk(k)[r * NX + c];
        }
        for (int t = tid; t < (N - 1) * NX * NU; t += nthr) {
          const int k = t / (NX * NU), r = (t / NU) % NX, c = t % NU;
          a.outB[bo + ((size_t)k * a.nx_max + r) * a.nu_max + c] = Bblk(k)[r * NU + c];
        }
        for (int t = tid; t < (N - 1) * NX; t += nthr) {
          const int k = t / NX, r = t % NX;
          a.oute[eo + (size_t)k * a.nx_max + r] = sm.e[k][r];
        }
        return;
      }
    } else {
      // Stage entry point: QP data supplied by the caller.
      const size_t ao = (size_t)sid * (a.N_max - 1) * a.nx_max * a.nx_max;
      const size_t bo = (size_t)sid * (a.N_max - 1) * a.nx_max * a.nu_max;
      for (int t = tid; t < (N - 1) * NX * NX; t += nthr) {
        const int k = t / (NX * NX), r = (t / NX) % NX, c = t % NX;
        Ablk(k)[r * NX + c] = a.inA[ao + ((size_t)k * a.nx_max + r) * a.nx_max + c];
      }
      for (int t = tid; t < (N - 1) * NX * NU; t += nthr) {
        const int k = t / (NX * NU), r = (t / NU) % NX, c = t % NU;
        Bblk(k)[r * NU + c] = a.inB[bo + ((size_t)k * a.nx_max + r) * a.nu_max + c];
      }
      for (int t = tid; t < N * G; t += nthr) {
        const int k = t / G, j = t % G;
        sm.qg[k][j] = j < NX ? a.inq[xoff + (size_t)k * a.nx_max + j] : 0.f;
        if (k < N - 1) {
          sm.e[k][j] = j < NX ? a.ine[(size_t)sid * (a.N_max - 1) * a.nx_max + (size_t)k * a.nx_max + j] : 0.f;
          if (j < 8) sm.rg[k][j] = j < NU ? a.inr[uoff + (size_t)k * a.nu_max + j] : 0.f;
        }
      }
      if (tid < G) sm.c0[tid] = tid < NX ? a.inc0[(size_t)sid * a.nx_max + tid] : 0.f;
    }
    __syncthreads();
    // The other parity's flag was last read before the previous iteration's
    // closing barrier; clear it for the next iteration.
    if (tid == 0) sm.bad[(it + 1) & 1] = 0;
    unpark();
    if constexpr (TS) {
      for (int t = tid; t < N; t += nthr) sm.mp0[t] += ts.mt[t];
      // Rewrite the QP in y_k = T_k^-1 x_k, and the warm-start multipliers
      // (lambda^ = T_k^T lambda).
#pragma unroll
      for (int p = 0; p < KPT; ++p) {
        const int k = slot + p * SLOTS;
        if (k < N) {
          const bool succ = k < N - 1;
          tip_rewrite<ND>(lane, succ, k == 0, h, ts.Lc[k], ts.Li[k], ts.Lc[succ ? k + 1 : k], Ablk(k) + lane * NX,
                          sm.e[k], sm.qg[k], sm.c0, ts.Jt[k], ts.pe[k], succ ? D.We : D.WeN, ts.tq[k]);
          lam[p] = (Real)tip_lambda<ND>(lane, true, ts.Lc[k], ts.Li[k], ts.tq[k], (double)lam[p]);
        }
      }
      __syncthreads();
    }
    if (clk) clk[1] = wall_clock64();

    int its = 0;
    bool capped = false;      // PCG stopped at its iteration limit
    bool xfail_any = false;   // some part of this solve gave up a wait
    if constexpr (kHalf) {
      // ================= 2. Schur rows and diagonal-block inverses, lane = row.
      // Rows of O_{k,k-1} and O_{k,k+1} (OffEuler; OffRows where the joint rows of A
      // are not the Euler step's: tip tracking, caller-given QP data).
      constexpr int KA = kLong ? 1 : KPT;
      double Am[KA][NX], Av[KA][ND], aj[KA];
      double Pd[KPT][NX];                                        // row of D_k^-1
      double gam[KPT], res[KPT], qown[KPT];
      // The A blocks as they are.
      const float *full = TS || (kLong ? KKT : a.mode == kModeKkt) ? Ablk(0) : nullptr;
      if constexpr (kLong) {
        for (int t = tid; t < PcgBufs<ND, KPT>::KH * G; t += nthr) (&sm.pcg.z[0][0])[t] = (&sm.pcg.v[0][0])[t] = 0.0;
        if (tid < 64) sm.pcg.red[tid] = 0.0;
      }
#pragma unroll
      for (int p = 0; p < KPT; ++p) {
        const int k = slot + p * SLOTS;
        double thr[NX];
        gam[p] = res[p] = qown[p] = 0.0;
#pragma unroll
        for (int m = 0; m < NX; ++m) {
          thr[m] = Pd[p][m] = 0.0;
          if constexpr (!kLong) Am[p][m] = 0.0;
        }
        if constexpr (!kLong) {
          aj[p] = 0.0;
#pragma unroll
          for (int m = 0; m < ND; ++m) Av[p][m] = 0.0;
        }
        if (k < N) {
          const double *Qik = (k < N - 1) ? sm.Qi : sm.Qni;
          if (lane < NX) {
            const int km = max(k - 1, 0);
            auto arow = [&](int m) -> double {
              if constexpr (kLong) {
                if (!full)
                  return lane < ND ? (m == lane ? 1.0 : 0.0) + (m == lane + ND ? (double)h : 0.0)
                                   : (double)sm.Av[km][max(lane - ND, 0)][m];
              }
              return (double)Ablk(km)[lane * NX + m];
            };
            qown[p] = Qik[lane];
            auto put = [&](int m, double x) {
              if constexpr (!kLong) Am[p][m] = x;
            };
            schur_knot<ND>(lane, k == 0, arow, put, Ablk(km), Bblk(km), sm.Qi, Qik, D.Ri, sm.c0, sm.e[km], sm.qg[k],
                           sm.qg[km], sm.rg[km], lam[p], thr, gam[p], res[p]);
            if constexpr (!kLong && !TS) {
              if (k < N - 1) {
                const float *A = Ablk(k);
                aj[p] = -qown[p] * (lane < ND ? 1.0 : (double)h);
#pragma unroll
                for (int m = 0; m < ND; ++m) Av[p][m] = -qown[p] * (double)A[(ND + m) * NX + lane];
              }
            }
          }
          invert_knot<ND, G == 16 && !TS>(lane, k == 0, sm.Qi, thr, sm.piv[slot], Pd[p]);
        }
      }
      if constexpr (kLong) __syncthreads();   // (the PCG's buffers are clear)
      if (clk) {
        clk[2] = wall_clock64();
        clk[3] = clk[2];
      }
      // ================= 3-5. Preconditioned CG, then the step dZ = -G^-1 (g - C^T
      // lambda): with the scaled columns, dx = -Q^-1 (q - lambda) + O_{k,k+1} lambda_{k+1}.
      const int max_it = a.pcg_max_iter > 0 ? a.pcg_max_iter : N * NX;
      const int slot_w = (__builtin_amdgcn_readfirstlane(tid) >> 6) * (64 / G);   // the wavefront's first lane group
      NoExchange none;
      auto pcg = [&](auto na, auto pipe, const auto &off) {
        its = pcg_half_sweeps<ND, KPT, na, pipe>(sm.pcg, tid, lane, slot, off, none, Pd, gam, res, lam, a.pcg_tol,
                                                 max_it, capped);
      };
      using std::integral_constant;
      const double q0 = lane < NX ? sm.Qi[lane] : 0.0;
      if constexpr (kLong) {
        int na = 0;
        for (int p = 0; p < KPT; ++p) na += slot_w + p * SLOTS < N ? 1 : 0;
        const OffLds<ND, KPT, KKT> off{sm.Av, full, qown, q0, (double)h, lane, slot, N};
        its = pcg_long<ND, KPT>(sm.pcg, tid, lane, slot, na, off, Pd, gam, res, lam, a.pcg_tol, max_it, capped);
      } else if (TS || full) {
        double Ac[KPT][NX];
#pragma unroll
        for (int p = 0; p < KPT; ++p) {
          const int k = slot + p * SLOTS;
          const float *A = full + (size_t)min(k, N - 2) * NX * NX;
#pragma unroll
          for (int m = 0; m < NX; ++m) Ac[p][m] = k < N - 1 && lane < NX ? -qown[p] * (double)A[m * NX + lane] : 0.0;
        }
        const OffRows<ND, KPT> off{Am, Ac};
        if (KPT > 1 && slot_w + SLOTS < N) pcg(integral_constant<int, KPT>{}, integral_constant<bool, !TS>{}, off);
        else if (slot_w < N) pcg(integral_constant<int, 1>{}, integral_constant<bool, !TS>{}, off);
        else pcg(integral_constant<int, 0>{}, integral_constant<bool, !TS>{}, off);
      } else if constexpr (!TS) {
        const OffEuler<ND, KPT> off{Am, Av, aj};
        if (KPT > 1 && slot_w + SLOTS < N) pcg(integral_constant<int, KPT>{}, std::true_type{}, off);
        else if (slot_w < N) pcg(integral_constant<int, 1>{}, std::true_type{}, off);
        else pcg(integral_constant<int, 0>{}, std::true_type{}, off);
      }
      if (clk) clk[4] = wall_clock64();
      // (z: last read before the last barrier of the PCG's loop.)
#pragma unroll
      for (int p = 0; p < KPT; ++p) sm.pcg.z[slot + p * SLOTS + 1][lane] = lam[p];
      __syncthreads();
#pragma unroll
      for (int p = 0; p < KPT; ++p) {
        const int k = slot + p * SLOTS;
        if (k < N && lane < NX) {
          double d = -qown[p] * ((double)sm.qg[k][lane] - lam[p]);
          const double *ln = sm.pcg.z[k + 2];
          if constexpr (kLong) {
            const OffLds<ND, KPT, KKT> off{sm.Av, full, qown, q0, (double)h, lane, slot, N};
            off.add_col(p, d, ln[lane], 0.0);
          } else if (TS || full) {
            if (k < N - 1) {
              const float *A = Ablk(k);
              double t = 0.0;
#pragma unroll
              for (int m = 0; m < NX; ++m) t += (double)A[m * NX + lane] * ln[m];
              d -= qown[p] * t;
            }
          } else {
            OffEuler<ND, KPT>{Am, Av, aj}.add_col(p, d, ln[lane], ln[lane < ND ? lane : lane - ND]);
          }
          const float dx = (float)d;
          sm.dX[k][lane] = dx;
          if (!isfinite(dx)) bad_flag = 1;
          if constexpr (TS) {
            if (lane < ND) ts.tq[k][lane] = d;
          }
          if (lane < NU && k < N - 1) {
            const float *B = Bblk(k);
            double su = (double)sm.rg[k][lane];
#pragma unroll
            for (int m = 0; m < NX; ++m) su += (double)B[m * NU + lane] * sm.pcg.z[k + 2][m];
            const float du = (float)(-D.Ri[lane] * su);
            sm.dU[k][lane] = du;
            if (!isfinite(du)) bad_flag = 1;
          }
        }
      }
    } else {
    // ================= 2. Schur complement rows and diagonal-block inverses.
    Real th[kThGlobal ? 1 : KPT][NX];   // row of the diagonal block theta_{k-1} (Q_0^-1 for k = 0)
    Real Am[KPT][NX];   // row `lane` of A_{k-1}: S~_{k,k-1} = -A_{k-1} Q_{k-1}^-1
    Real Ac[KPT][NX];   // column `lane` of A_k: S~_{k,k+1} = -Q_k^-1 A_k^T
    Real gam[KPT];
    Real qown[KPT];       // Q_k^-1 at (lane, lane)
    Real Pd[KPT][NX];     // row of the inverse diagonal block (preconditioner)
#pragma unroll
    for (int p = 0; p < KPT; ++p) {
      const int k = slot + p * SLOTS;
      const bool valid = k < N && lane < NX;
      Real thr[NX];
#pragma unroll
      for (int m = 0; m < NX; ++m) {
        thr[m] = 0;
        Am[p][m] = 0.f;
        Ac[p][m] = 0.f;
        Pd[p][m] = 0;
      }
      gam[p] = 0;
      qown[p] = 0;
      if (valid) {
        const double *Qik = (k < N - 1) ? sm.Qi : sm.Qni;
        qown[p] = (Real)Qik[lane];
        if (k == 0) {
#pragma unroll
          for (int m = 0; m < NX; ++m) thr[m] = (m == lane) ? (Real)sm.Qi[lane] : (Real)0;
          gam[p] = (Real)sm.c0[lane] + (Real)sm.Qi[lane] * (Real)sm.qg[0][lane];
        } else {
          const int km = k - 1;
          const float *A = Ablk(km);
          const float *B = Bblk(km);
          Real ArQ[NX], BrR[NU];
#pragma unroll
          for (int m = 0; m < NX; ++m) {
            const float arow = A[lane * NX + m];
            Am[p][m] = arow;
            ArQ[m] = (Real)arow * (Real)sm.Qi[m];
          }
#pragma unroll
          for (int m = 0; m < NU; ++m) BrR[m] = (Real)B[lane * NU + m] * (Real)D.Ri[m];
#pragma unroll
          for (int c = 0; c < NX; ++c) {
            Real t = (c == lane) ? (Real)Qik[lane] : (Real)0;
#pragma unroll
            for (int m = 0; m < NX; ++m) t += ArQ[m] * (Real)A[c * NX + m];
#pragma unroll
            for (int m = 0; m < NU; ++m) t += BrR[m] * (Real)B[c * NU + m];
            thr[c] = t;
          }
          Real z = (Real)sm.e[km][lane] + (Real)Qik[lane] * (Real)sm.qg[k][lane];
#pragma unroll
          for (int m = 0; m < NX; ++m) z -= ArQ[m] * (Real)sm.qg[km][m];
#pragma unroll
          for (int m = 0; m < NU; ++m) z -= BrR[m] * (Real)sm.rg[km][m];
          gam[p] = z;
        }
        if (k < N - 1) {
          const float *A = Ablk(k);
#pragma unroll
          for (int m = 0; m < NX; ++m) Ac[p][m] = A[m * NX + lane];
        }
      }
      // Inverse of the diagonal block: Gauss-Jordan inside the lane group
      // (the block is SPD, so no pivoting is needed).
      if (k < N) {
        if (k == 0) {
          const Real d0 = lane < NX ? (Real)1 / (Real)sm.Qi[lane] : (Real)0;
#pragma unroll
          for (int m = 0; m < NX; ++m) Pd[p][m] = (m == lane) ? d0 : (Real)0;
        } else {
          // T: the arithmetic of the elimination (Real, or double when the
          // all-FP32 variant is asked for an FP64 block inverse).
          auto gauss_jordan = [&](auto tag) {
            using T = decltype(tag);
            T row[NX];
#pragma unroll
            for (int c = 0; c < NX; ++c) row[c] = (T)thr[c];
            if constexpr (std::is_same_v<T, double> && G == 16 && !TS) {
              gj_dpp<NX>(row, lane, std::make_integer_sequence<int, NX>{});
            } else {
#pragma unroll
            for (int pv = 0; pv < NX; ++pv) {
              if (lane == pv) {
#pragma unroll
                for (int c = 0; c < NX; ++c) sm.piv[slot][c] = (double)row[c];
              }
              wave_sync();
              T prow[NX];
#pragma unroll
              for (int c = 0; c < NX; ++c) prow[c] = (T)sm.piv[slot][c];
              wave_sync();
              const T pinv = (T)1 / prow[pv];
              if (lane == pv) {
#pragma unroll
                for (int c = 0; c < NX; ++c) row[c] = (c == pv) ? pinv : row[c] * pinv;
              } else {
                const T f = row[pv] * pinv;
#pragma unroll
                for (int c = 0; c < NX; ++c) row[c] = (c == pv) ? -f : row[c] - f * prow[c];
              }
            }
            }
#pragma unroll
            for (int c = 0; c < NX; ++c) Pd[p][c] = (Real)row[c];
          };
          if (sizeof(Real) == 4 && a.fp64_inv) gauss_jordan(double{});
          else gauss_jordan(Real{});
        }
        if (lane < NX) {
          float *Dk = Dblk(k) + lane * NX;
#pragma unroll
          for (int c = 0; c < NX; ++c) Dk[c] = (float)Pd[p][c];
        }
      }
      if constexpr (kThGlobal) {
        if (valid) {
          Real *Tk = Tblk(k) + lane * NX;
#pragma unroll
          for (int c = 0; c < NX; ++c) Tk[c] = thr[c];
        }
      } else {
#pragma unroll
        for (int c = 0; c < NX; ++c) th[p][c] = thr[c];
      }
    }
    __syncthreads();
    if (clk) clk[2] = wall_clock64();

    // ================= 3. Off-diagonal blocks of the stair preconditioner.
    // Explicit form (the all-FP32 variant with one knot per lane group): the
    // lanes of knot k (k >= 1) form row `lane` of
    //   P_{k,k-1} = -D_k^-1 phi_{k-1} D_{k-1}^-1,  phi_{k-1} = -A_{k-1} Q_{k-1}^-1,
    // keep it, and publish it so that knot k-1 can read its column. Either
    // form is a fixed linear operator, as the pipelined recurrences require.
    // With kFactP (several knots per lane group, where registers are short, and
    // tip tracking) the off-diagonal blocks are not formed:
    // P w = D^-1 (w - O D^-1 w), with O the off-diagonal blocks of S~ that the
    // S~ product already holds.
    constexpr bool kFactP = KPT > 1 || TS;
    constexpr int KP = kFactP ? 1 : KPT;
    Real Pm[KP][NX], Pp[KP][NX], Pdf[KPT][NX];
#pragma unroll
    for (int p = 0; p < KPT; ++p) {
#pragma unroll
      for (int m = 0; m < NX; ++m) Pdf[p][m] = Pd[p][m];
    }
    if constexpr (!kFactP) {
#pragma unroll
    for (int p = 0; p < KPT; ++p) {
      const int k = slot + p * SLOTS;
      const bool valid = k < N && lane < NX;
#pragma unroll
      for (int m = 0; m < NX; ++m) {
        Pm[p][m] = 0.f;
        Pp[p][m] = 0.f;
      }
      if (valid && k >= 1) {
        const float *A = Ablk(k - 1);
        const float *Dm = Dblk(k - 1);
        float t[NX];
#pragma unroll
        for (int c = 0; c < NX; ++c) {
          float s = 0.f;
#pragma unroll
          for (int m = 0; m < NX; ++m) s += (float)Pd[p][m] * A[m * NX + c];
          t[c] = s * (float)sm.Qi[c];   // = -(D_k^-1 phi_{k-1})[lane][c]
        }
        float *Po = Pblk(k - 1) + lane * NX;
#pragma unroll
        for (int c2 = 0; c2 < NX; ++c2) {
          float s = 0.f;
#pragma unroll
          for (int c = 0; c < NX; ++c) s += t[c] * Dm[c * NX + c2];
          Pm[p][c2] = s;
          Po[c2] = s;
        }
      }
    }
    __syncthreads();
#pragma unroll
    for (int p = 0; p < KPT; ++p) {
      const int k = slot + p * SLOTS;
      if (k < N - 1 && lane < NX) {
        const float *Po = Pblk(k);
#pragma unroll
        for (int m = 0; m < NX; ++m) Pp[p][m] = Po[m * NX + lane];   // P_{k,k+1} = P_{k+1,k}^T
      }
    }
    }  // !kFactP

    if (clk) clk[3] = wall_clock64();
    // ================= 4. PCG on S~ lambda = gamma~: the standard (Hestenes-Stiefel)
    // arrangement, whose directly computed p^T S~ p tolerates the rounding of FP32
    // vectors.
    // Split solve: this part's rows only, until the multipliers are gathered.
    bool xon = split;
    auto own = [&](int p) { return !xon || (p >> psh) == part; };
    unsigned long long *xb = split ? a.xch + D.xch_off : nullptr;
    const int xspin = a.xspin > 0 ? a.xspin : kXSpin;
    auto xtag = [&](unsigned e) { return ((a.epoch & 0xffffu) << 16) | (e & 0xffffu); };
    auto xslot = [&](int q, unsigned e) { return xb + (size_t)q * kXPart + (size_t)(e % kXSlots) * kXSlot; };
    const int kf = (part << psh) * SLOTS;                        // own knots kf..kl (none when kf >= N)
    const int kl = min(kf + (SLOTS << psh), N) - 1;
    const bool has_l = split && part > 0 && kf < N;              // a part on the left / the right
    const bool has_r = split && kl + 1 < N;
    // Halo rows: the first own knot's row of vl goes to the left part, the last
    // one's of vr to the right part; the neighbours' rows land in vr[kf - 1]
    // and vl[kl + 1], read only by the lane groups that receive them.
    // (Published where the rows are formed, in share_S and prepare_P, for
    // the exchange that follows them: number xe.)
    auto xhalo_put_row = [&](int k, double left, double right) {
      if (lane < NX) {
        if (has_l && k == kf) xput(xslot(part, xe) + 2 * lane, xtag(xe), left);
        if (has_r && k == kl) xput(xslot(part, xe) + 32 + 2 * lane, xtag(xe), right);
      }
    };
    auto xhalo_get = [&](unsigned e, Real (*vl)[G], Real (*vr)[G]) {
      const bool dead = sm.xfail != 0;
      if (lane < NX) {
        double v;
        if (has_l && slot == 0) {
          if (!xget(xslot(part - 1, e) + 32 + 2 * lane, xtag(e), dead, xspin, v)) sm.xfail = 1;
          vr[kf - 1][lane] = (Real)v;
        }
        if (has_r && slot == kl % SLOTS) {
          if (!xget(xslot(part + 1, e) + 2 * lane, xtag(e), dead, xspin, v)) sm.xfail = 1;
          vl[kl + 1][lane] = (Real)v;
        }
      }
      wave_sync();
    };
    // Sums over the parts (fixed order) of three partials that every lane holds.
    auto xsum_put = [&](unsigned e, double s0, double s1, double s2) {
      if (tid < 3) xput(xslot(part, e) + 64 + 2 * tid, xtag(e), tid == 0 ? s0 : (tid == 1 ? s1 : s2));
    };
    // Halo rows and sums of one exchange, all words polled together.
    auto xhalo_sum_get = [&](unsigned e, bool halo, Real (*vl)[G], Real (*vr)[G], double &s0, double &s1,
                             double &s2) {
      const bool dead = sm.xfail != 0;
      const int l = tid & 63;
      const bool hl = halo && has_l && slot == 0 && lane < NX;
      const bool hr = halo && has_r && slot == kl % SLOTS && lane < NX;
      unsigned long long *wh = hl ? xslot(part - 1, e) + 32 + 2 * lane : (hr ? xslot(part + 1, e) + 2 * lane : nullptr);
      unsigned long long *ws = l < 3 * nparts ? xslot(l / 3, e) + 64 + 2 * (l % 3) : nullptr;
      double vh = 0.0, v = 0.0;
      if (wh || ws) {
        bool ok;
        if (wh && ws) ok = xget2(wh, ws, xtag(e), dead, xspin, vh, v);
        else if (wh) ok = xget(wh, xtag(e), dead, xspin, vh);
        else ok = xget(ws, xtag(e), dead, xspin, v);
        if (!ok) sm.xfail = 1;
      }
      if (hl) vr[kf - 1][lane] = (Real)vh;
      if (hr) vl[kl + 1][lane] = (Real)vh;
      wave_sync();
      if (nparts == 2) {
        s0 = lane_val(v, 0) + lane_val(v, 3);
        s1 = lane_val(v, 1) + lane_val(v, 4);
        s2 = lane_val(v, 2) + lane_val(v, 5);
      } else {
        s0 = (lane_val(v, 0) + lane_val(v, 3)) + (lane_val(v, 6) + lane_val(v, 9));
        s1 = (lane_val(v, 1) + lane_val(v, 4)) + (lane_val(v, 7) + lane_val(v, 10));
        s2 = (lane_val(v, 2) + lane_val(v, 5)) + (lane_val(v, 8) + lane_val(v, 11));
      }
    };
    auto xhalo = [&](Real (*vl)[G], Real (*vr)[G]) {
      xhalo_get(xe, vl, vr);
      ++xe;
    };
    // Sums over the parts of three workgroup totals (no halo rows).
    auto xsums = [&](double &s0, double &s1, double &s2) {
      xsum_put(xe, s0, s1, s2);
      xhalo_sum_get(xe, false, sm.pv, sm.sv, s0, s1, s2);
      ++xe;
    };
    // Every part's multipliers to every part (after the PCG).
    auto xlam = [&]() {
      const unsigned e = xe++;
#pragma unroll
      for (int p = 0; p < KPT; ++p)
        if ((p >> psh) == part && slot + p * SLOTS < N && lane < NX)
          xput(xb + (size_t)p * kXPart + kXSlots * kXSlot + 2 * (slot * G + lane), xtag(e), (double)lam[p]);
      const bool dead = sm.xfail != 0;
#pragma unroll
      for (int p = 0; p < KPT; ++p) {
        if ((p >> psh) != part && slot + p * SLOTS < N && lane < NX) {
          double v;
          if (!xget(xb + (size_t)p * kXPart + kXSlots * kXSlot + 2 * (slot * G + lane), xtag(e), dead, xspin, v))
            sm.xfail = 1;
          lam[p] = (Real)v;
        }
      }
    };
    auto share_S = [&](const Real *vals) {   // operand of S~: vals and Q^-1 vals
#pragma unroll
      for (int p = 0; p < KPT; ++p) {
        const int k = slot + p * SLOTS;
        if (k < N && own(p)) {
          const bool valid = lane < NX;
          sm.pv[k][lane] = valid ? vals[p] : (Real)0;
          sm.sv[k][lane] = valid ? qown[p] * vals[p] : (Real)0;
          if (xon) xhalo_put_row(k, (double)vals[p], (double)(qown[p] * vals[p]));
        }
      }
    };
    auto share_P = [&](const Real *vals, Real (*buf)[G]) {
#pragma unroll
      for (int p = 0; p < KPT; ++p) {
        const int k = slot + p * SLOTS;
        if (k < N && own(p)) buf[k][lane] = (lane < NX) ? vals[p] : (Real)0;
      }
    };
    // With one knot per lane group, block-row products accumulate in two
    // interleaved partial sums per block (even and odd columns), so that the FMA
    // chains are short and independent; with more knots the extra accumulators
    // would cost registers (spills), so the odd columns fold into the even sums.
    constexpr bool kSplit = (KPT == 1);
    auto apply_S = [&](int p) -> Real {
      const int k = slot + p * SLOTS;
      if constexpr (kSplit) {
        Real d0 = 0, d1 = 0, l0 = 0, l1 = 0, u0 = 0, u1 = 0;
#pragma unroll
        for (int m = 0; m < NX; m += 2) {
          d0 += th[p][m] * sm.pv[k][m];
          d1 += th[p][m + 1] * sm.pv[k][m + 1];
        }
        if (k > 0) {
#pragma unroll
          for (int m = 0; m < NX; m += 2) {
            l0 += Am[p][m] * sm.sv[k - 1][m];
            l1 += Am[p][m + 1] * sm.sv[k - 1][m + 1];
          }
        }
        if (k < N - 1) {
#pragma unroll
          for (int m = 0; m < NX; m += 2) {
            u0 += Ac[p][m] * sm.pv[k + 1][m];
            u1 += Ac[p][m + 1] * sm.pv[k + 1][m + 1];
          }
        }
        return ((d0 + d1) - (l0 + l1)) - qown[p] * (u0 + u1);
      } else {
        Real acc = 0;
#pragma unroll
        for (int m = 0; m < NX; ++m) {
          if constexpr (kThGlobal) acc += Tblk(k)[lane * NX + m] * sm.pv[k][m];
          else acc += th[p][m] * sm.pv[k][m];
        }
        if (k > 0) {
#pragma unroll
          for (int m = 0; m < NX; ++m) acc -= Am[p][m] * sm.sv[k - 1][m];
        }
        if (k < N - 1) {
          Real t = 0;
#pragma unroll
          for (int m = 0; m < NX; ++m) t += Ac[p][m] * sm.pv[k + 1][m];
          acc -= qown[p] * t;
        }
        return acc;
      }
    };
    auto apply_P = [&](int p, Real (*buf)[G]) -> Real {
      const int k = slot + p * SLOTS;
      Real acc = 0;
      if constexpr (!kFactP) {
        Real d0 = 0, d1 = 0, l0 = 0, l1 = 0, u0 = 0, u1 = 0;
#pragma unroll
        for (int m = 0; m < NX; m += 2) {
          d0 += (Real)Pdf[p][m] * buf[k][m];
          d1 += (Real)Pdf[p][m + 1] * buf[k][m + 1];
        }
        if (k > 0) {
#pragma unroll
          for (int m = 0; m < NX; m += 2) {
            l0 += (Real)Pm[p][m] * buf[k - 1][m];
            l1 += (Real)Pm[p][m + 1] * buf[k - 1][m + 1];
          }
        }
        if (k < N - 1) {
#pragma unroll
          for (int m = 0; m < NX; m += 2) {
            u0 += (Real)Pp[p][m] * buf[k + 1][m];
            u1 += (Real)Pp[p][m + 1] * buf[k + 1][m + 1];
          }
        }
        acc = (d0 + d1) + ((l0 + l1) + (u0 + u1));
      }
      return acc;
    };
    // Factored preconditioner, two halves around the workgroup barrier that
    // publishes the operand (the explicit form publishes it with share_P):
    //   prepare: z_k = D_k^-1 v_k (own knot, exchanged inside the lane group),
    //            published with Q_k^-1 z_k in rv / gv;
    //   finish:  t_k = v_k - (O z)_k, then (P v)_k = D_k^-1 t_k.
    auto group_dinv = [&](int p, Real x) -> Real {   // row `lane` of D_k^-1 times the group's x
      const int k = slot + p * SLOTS;
      Real acc = 0;
      sm.tv[k][lane] = (lane < NX) ? x : (Real)0;
      wave_sync();
#pragma unroll
      for (int m = 0; m < NX; ++m) acc += Pdf[p][m] * sm.tv[k][m];
      wave_sync();
      return acc;
    };
    auto prepare_P = [&](const Real *vals) {
#pragma unroll
      for (int p = 0; p < KPT; ++p) {
        const int k = slot + p * SLOTS;
        if (k < N && own(p)) {
          const Real z = group_dinv(p, vals[p]);
          sm.rv[k][lane] = (lane < NX) ? z : (Real)0;
          sm.gv[k][lane] = (lane < NX) ? qown[p] * z : (Real)0;
          if (xon) xhalo_put_row(k, (double)z, (double)(qown[p] * z));
        }
      }
    };
    auto finish_P = [&](int p, Real v) -> Real {
      const int k = slot + p * SLOTS;
      Real oz = 0;   // (O z)_k at row `lane`
      if (k > 0) {
#pragma unroll
        for (int m = 0; m < NX; ++m) oz -= Am[p][m] * sm.gv[k - 1][m];
      }
      if (k < N - 1) {
        Real t = 0;
#pragma unroll
        for (int m = 0; m < NX; ++m) t += Ac[p][m] * sm.rv[k + 1][m];
        oz -= qown[p] * t;
      }
      return group_dinv(p, v - oz);
    };
    auto row_valid = [&](int p) { return (slot + p * SLOTS) < N && lane < NX && own(p); };

    // r = gamma~ - S~ lambda, u = P r, w = S~ u; eta_ref = gamma~^T P gamma~.
    Real r[KPT], u[KPT], w[KPT], vp[KPT];
    share_S(lam);
    __syncthreads();
    if (xon) xhalo(sm.pv, sm.sv);
#pragma unroll
    for (int p = 0; p < KPT; ++p) r[p] = row_valid(p) ? gam[p] - apply_S(p) : (Real)0;
    Real Pgam[KPT];   // P gamma~, for the reference norm
    if constexpr (kFactP) {
      prepare_P(r);
      __syncthreads();
      if (xon) xhalo(sm.rv, sm.gv);
#pragma unroll
      for (int p = 0; p < KPT; ++p) u[p] = row_valid(p) ? finish_P(p, r[p]) : (Real)0;
      __syncthreads();
      prepare_P(gam);
      __syncthreads();
      if (xon) xhalo(sm.rv, sm.gv);
#pragma unroll
      for (int p = 0; p < KPT; ++p) Pgam[p] = row_valid(p) ? finish_P(p, gam[p]) : (Real)0;
    } else {
      share_P(r, sm.rv);
      share_P(gam, sm.gv);
      __syncthreads();
#pragma unroll
      for (int p = 0; p < KPT; ++p) {
        u[p] = row_valid(p) ? apply_P(p, sm.rv) : (Real)0;
        Pgam[p] = row_valid(p) ? apply_P(p, sm.gv) : (Real)0;
      }
    }
    Real eta_ref = 0;
#pragma unroll
    for (int p = 0; p < KPT; ++p) eta_ref += gam[p] * Pgam[p];
    const int max_it = a.pcg_max_iter > 0 ? a.pcg_max_iter : N * NX;
    Real gma = 0, stop = 0;
    {
      // Acc: the accumulation type of the inner products.
      auto run = [&](auto tag) {
        using Acc = decltype(tag);
        Acc sums[3] = {0, 0, 0};
#pragma unroll
        for (int p = 0; p < KPT; ++p) {
          sums[0] += (Acc)r[p] * (Acc)u[p];
          sums[2] += (Acc)gam[p] * (Acc)Pgam[p];
          vp[p] = u[p];
        }
        block_sum<3>(sm.red, redbuf, sums);
        if (xon) {
          double t0 = (double)sums[0], t1 = (double)sums[1], t2 = (double)sums[2];
          xsums(t0, t1, t2);
          sums[0] = (Acc)t0;
          sums[2] = (Acc)t2;
        }
        Acc g = sums[0];
        const Acc stop_a = (Acc)a.pcg_tol * (Acc)a.pcg_tol * sums[2];
        while (g > stop_a && its < max_it) {
          share_S(vp);
          __syncthreads();
          if (xon) xhalo(sm.pv, sm.sv);
          Acc pw[1] = {0};
#pragma unroll
          for (int p = 0; p < KPT; ++p) {
            w[p] = row_valid(p) ? apply_S(p) : (Real)0;
            pw[0] += (Acc)vp[p] * (Acc)w[p];
          }
          block_sum<1>(sm.red, redbuf, pw);
          if (xon) {
            double t0 = (double)pw[0], t1 = 0.0, t2 = 0.0;
            xsums(t0, t1, t2);
            pw[0] = (Acc)t0;
          }
          const Real alpha = (Real)div_pcg(g, pw[0]);
#pragma unroll
          for (int p = 0; p < KPT; ++p) {
            lam[p] += alpha * vp[p];
            r[p] -= alpha * w[p];
          }
          if constexpr (kFactP) prepare_P(r);
          else share_P(r, sm.rv);
          __syncthreads();
          if (xon) xhalo(sm.rv, sm.gv);
          Acc rz[1] = {0};
#pragma unroll
          for (int p = 0; p < KPT; ++p) {
            if constexpr (kFactP) u[p] = row_valid(p) ? finish_P(p, r[p]) : (Real)0;
            else u[p] = row_valid(p) ? apply_P(p, sm.rv) : (Real)0;
            rz[0] += (Acc)r[p] * (Acc)u[p];
          }
          block_sum<1>(sm.red, redbuf, rz);
          if (xon) {
            double t0 = (double)rz[0], t1 = 0.0, t2 = 0.0;
            xsums(t0, t1, t2);
            rz[0] = (Acc)t0;
          }
          const Real beta = (Real)div_pcg(rz[0], g);
          g = rz[0];
#pragma unroll
          for (int p = 0; p < KPT; ++p) vp[p] = u[p] + beta * vp[p];
          ++its;
        }
        // Only the convergence test outlives the loop (status bits).
        gma = (g > stop_a) ? (Real)1 : (Real)0;
        stop = 0;
      };
      if (a.fp64_dot) run(double{});
      else run(float{});
    }
    if (xon) {
      xlam();
      xon = false;
      // Every part's failure flag to every part: a part that gave up still
      // publishes (without waiting), so a writer that did not give up learns
      // that the rows it received were not the other parts' results.
      __syncthreads();
      double f0 = sm.xfail ? 1.0 : 0.0, f1 = 0.0, f2 = 0.0;
      xsums(f0, f1, f2);
      xfail_any = f0 != 0.0;
    }
    capped = gma > stop;
    if (clk) clk[4] = wall_clock64();

    // ================= 5. Step recovery dZ = -G^-1 (g - C^T lambda).
    share_S(lam);
    __syncthreads();
#pragma unroll
    for (int p = 0; p < KPT; ++p) {
      const int k = slot + p * SLOTS;
      if (k < N && lane < NX) {
        Real sx = (Real)sm.qg[k][lane] - lam[p];
        if (k < N - 1) {
#pragma unroll
          for (int m = 0; m < NX; ++m) sx += Ac[p][m] * sm.pv[k + 1][m];
        }
        const float dx = (float)(-qown[p] * sx);
        sm.dX[k][lane] = dx;
        if (!isfinite(dx)) bad_flag = 1;
        if constexpr (TS) {
          if (lane < ND) ts.tq[k][lane] = (double)(-qown[p] * sx);
        }
        if (lane < NU && k < N - 1) {
          const float *B = Bblk(k);
          Real su = (Real)sm.rg[k][lane];
#pragma unroll
          for (int m = 0; m < NX; ++m) su += (Real)B[m * NU + lane] * sm.pv[k + 1][m];
          const float du = (float)(-(Real)D.Ri[lane] * su);
          sm.dU[k][lane] = du;
          if (!isfinite(du)) bad_flag = 1;
        }
      }
    }
    }  // !kHalf
    unsigned status = capped ? GATO_ST_PCG_MAXITER : 0u;
    if constexpr (TS) {
      // Back to x: dx_k = T_k dy_k (joint rows L_k^-T dy), lambda = T_k^-T lambda^.
#pragma unroll
      for (int p = 0; p < KPT; ++p) {
        const int k = slot + p * SLOTS;
        if (k < N) {
          const double *Lk = ts.Lc[k];
          const double *Lik = ts.Li[k];
          wave_sync();
          double t = 0.0;
          if (lane < ND) {
#pragma unroll
            for (int m = 0; m < ND; ++m)
              if (m >= lane) t += Lik[tri(m, lane)] * ts.tq[k][m];
          }
          wave_sync();
          if (lane < ND) {
            const float dx = (float)t;
            sm.dX[k][lane] = dx;
            if (!isfinite(dx)) bad_flag = 1;
            ts.tq[k][lane] = (double)lam[p];
          }
          wave_sync();
          if (lane < ND) {
            double l = 0.0;
#pragma unroll
            for (int m = 0; m < ND; ++m)
              if (m <= lane) l += Lk[tri(lane, m)] * ts.tq[k][m];
            lam[p] = (Real)l;
          }
        }
      }
    }
    if (a.mode == kModeKkt) {
      __syncthreads();
#pragma unroll
      for (int p = 0; p < KPT; ++p) {
        const int k = slot + p * SLOTS;
        if (k < N && lane < NX) {
          a.outdX[xoff + (size_t)k * a.nx_max + lane] = sm.dX[k][lane];
          a.outlam[xoff + (size_t)k * a.nx_max + lane] = (double)lam[p];
          if (lane < NU && k < N - 1) a.outdU[uoff + (size_t)k * a.nu_max + lane] = sm.dU[k][lane];
        }
      }
      if (tid == 0 && a.outits) a.outits[sid] = its;
      return;
    }
    park();
    __syncthreads();
    if (clk) clk[5] = wall_clock64();

    // ================= 6. Line search over alpha_i = beta^-i (Eqs. (3), (7)).
    // (The biases go through the space of the A blocks, whose last reads, in phase 5
    // with tip tracking and caller-given data, the barrier above orders before it.)
    float *kpt_bias = nullptr;
    if constexpr (KPT == 1) {
      static_assert(kBlock / 2 * ND <= BS::LB * NX * NX && BS::kLds, "biases of the trial knots");
      kpt_bias = &sm.A[0][0];
    }
    if (const int i = ls_trials<ND, TS, KPT == 1>(sm, a, sid, D.We, ts.pr, kpt_bias, tid, nthr, n_alpha, 0, N - 1, h);
        i < n_alpha) {
      const float al = sm.alpha[i];
      float cost = 0.f, viol = 0.f;
      for (int j = 0; j < NX; ++j) {
        const float d = (sm.X[N - 1][j] + al * sm.dX[N - 1][j]) - sm.xg[j];
        cost += 0.5f * D.Wn[j] * d * d;
        viol += fabsf(sm.xs[j] - (sm.X[0][j] + al * sm.dX[0][j]));
      }
      if constexpr (TS) {
        float q[ND], pt[3];
#pragma unroll
        for (int j = 0; j < ND; ++j) q[j] = sm.X[N - 1][j] + al * sm.dX[N - 1][j];
        tip_position<ND>(D.chain, q, pt);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          const float d = pt[c] - ts.pr[N - 1][c];
          cost += 0.5f * D.WeN[c] * d * d;
        }
      }
      sm.mp[i][N - 1] = (double)cost + (double)a.mu * (double)viol;
    }
    __syncthreads();
    if (tid <= n_alpha) {
      double sum = 0.0;
      for (int k = 0; k < N; ++k) sum += (tid == n_alpha) ? sm.mp0[k] : sm.mp[tid][k];
      sm.merit[tid] = sum;
    }
    __syncthreads();
    int best = -1;
    for (int i = 0; i < n_alpha; ++i) {
      const double m = sm.merit[i];
      if (isfinite(m) && (best < 0 || m < sm.merit[best])) best = i;
    }
    const bool bad = bad_flag != 0 || best < 0;
    if (bad) status |= GATO_ST_NONFINITE;
    else if (!(sm.merit[best] < sm.merit[n_alpha])) status |= GATO_ST_NO_DESCENT;
    const double rho_used = rho;
    if (a.rho_adapt) rho = (status & (GATO_ST_NONFINITE | GATO_ST_NO_DESCENT)) ? fmin(2.0 * rho, 1e8) : rho / 3.0;
    const float al = bad ? 0.f : sm.alpha[best];
    if (!bad) {
      for (int t = tid; t < N * G; t += nthr) {
        const int k = t / G, j = t % G;
        sm.X[k][j] += al * sm.dX[k][j];
        if (k < N - 1 && j < 8) sm.U[k][j] += al * sm.dU[k][j];
      }
    }
    if (split && (sm.xfail || xfail_any)) status |= GATO_ST_EXCHANGE;
    if (tid == 0 && a.stats && writer) {
      gato_solve_stats st;
      st.merit0 = (float)sm.merit[n_alpha];
      st.merit = bad ? (float)sm.merit[n_alpha] : (float)sm.merit[best];
      st.alpha = al;
      st.pcg_iters = its;
      st.status = status;
      st.rho = (float)rho_used;
      a.stats[(size_t)rid * a.stats_stride + it] = st;
    }
    __syncthreads();
    if (clk) {
      clk[6] = wall_clock64();
      clk[7] = clock64() - cyc0;
    }
  }

  // ---- Write back the iterate, the warm-start multipliers and the adapted damping.
  const int lane = lane0, slot = slot0;
  unpark();
  if (a.mode == kModeSqp && writer) {
    if (a.rho_adapt && tid == 0) a.rho[sid] = rho;
    const size_t rxo = (size_t)blockIdx.x * a.N_max * a.nx_max;
    const size_t ruo = (size_t)blockIdx.x * (a.N_max - 1) * a.nu_max;
    for (int t = tid; t < N * G; t += nthr) {
      const int k = t / G, j = t % G;
      if (j < NX) {
        a.X[xoff + (size_t)k * a.nx_max + j] = sm.X[k][j];
        if (a.Xout) a.Xout[rxo + (size_t)k * a.nx_max + j] = sm.X[k][j];
        if (a.x1out && k == 1) a.x1out[(size_t)blockIdx.x * a.nx_max + j] = sm.X[k][j];
      }
      if (k < N - 1 && j < NU) {
        a.U[uoff + (size_t)k * a.nu_max + j] = sm.U[k][j];
        if (a.Uout) a.Uout[ruo + (size_t)k * a.nu_max + j] = sm.U[k][j];
        if (a.u0out && k == 0) a.u0out[(size_t)blockIdx.x * a.nu_max + j] = sm.U[k][j];
      }
    }
#pragma unroll
    for (int p = 0; p < KPT; ++p) {
      const int k = slot + p * SLOTS;
      if (k < N && lane < NX) gL[k * a.nx_max + lane] = (double)lam[p];
    }
  }
}

template <int ND, int KPT, class Real, bool TS = false, bool SPLIT = false>
__global__ __launch_bounds__(kBlock) void sqp_kernel(KArgs a) {
  constexpr size_t kOne = smem_bytes<ND, KPT, Real, TS>();
  constexpr size_t kPart = SPLIT && sizeof(Real) == 8 ? long_part_bytes<ND>() : 0;
  constexpr size_t kBytes = kOne > kPart ? kOne : kPart;
  static_assert(kBytes <= 160 * 1024, "LDS of one workgroup exceeds 160 KB");
  static_assert(KPT != 1 || TS || sizeof(Real) == 4 || 2 * kBytes <= 160 * 1024, "block_threads: two workgroups to a CU");
  __shared__ __align__(16) char smem[kBytes];
  int sid = a.order ? a.order[blockIdx.x] : a.sid_base + (int)blockIdx.x;
  int part = 0;
  if constexpr (SPLIT) {
    if (a.split) {
      part = (int)((unsigned)sid >> 24);
      sid &= 0xffffff;
    }
  }
  if (sid < 0 || sid >= a.M) return;   // a caller-provided slot out of range: nothing to do
  sqp_solve<ND, KPT, Real, TS, SPLIT>(a, sid, part, smem);
}

// Long solves of caller-given QP data (FP64).
template <int ND>
__global__ __launch_bounds__(kBlock) void kkt_kernel(KArgs a) {
  __shared__ __align__(16) char smem[smem_bytes<ND, 4, double, false>()];
  const int sid = a.order ? a.order[blockIdx.x] : a.sid_base + (int)blockIdx.x;
  if (sid < 0 || sid >= a.M) return;
  sqp_solve<ND, 4, double, false, false, true>(a, sid, 0, smem);
}

// Mixed-shape kernel: every workgroup reads its solve's (n, kpt) and runs the
// matching specialisation, so a batch of uneven DoF and horizon is one launch.
// The LDS footprint is the largest specialisation's, and the workgroup has kBlock
// threads: one workgroup per CU, where a one-shape launch of short horizons runs two
// (block_threads). (For 3 DoF, two knots per 8-lane group already cover the maximum
// horizon; the task-space variant is compiled for one and two knots per group, and
// its long solves (6-7 DoF, N > 64) run only split, in the part-local form; long
// solves of caller-given QP data have kernels of their own.)
template <class Real, bool TS, bool SPLIT>
constexpr size_t mixed_smem_bytes() {
  size_t m = SPLIT && !TS && sizeof(Real) == 8 ? long_part_bytes<7>() : 0;
  const size_t s[] = {smem_bytes<3, 1, Real, TS>(), smem_bytes<3, 2, Real, TS>(),
                      smem_bytes<6, 1, Real, TS>(), smem_bytes<6, 2, Real, TS>(),
                      TS ? part_smem_bytes<6, 1, true>() : smem_bytes<6, 4, Real, false>(),
                      smem_bytes<7, 1, Real, TS>(), smem_bytes<7, 2, Real, TS>(),
                      TS ? part_smem_bytes<7, 1, true>() : smem_bytes<7, 4, Real, false>()};
  for (size_t v : s) m = v > m ? v : m;
  return m;
}

// A long task-space solve runs only as the four parts of a split SQP launch
// in FP64 (the host builds no other launch of one).
__device__ __forceinline__ bool task_split_ok(const KArgs &a, const SolveDesc &D, int part) {
  return a.split == kXParts && a.mode == kModeSqp && !a.by_block && D.xch_off >= 0 && part >= 0 && part < kXParts;
}

template <class Real, bool TS = false, bool SPLIT = false>
__global__ __launch_bounds__(kBlock) void sqp_mixed_kernel(KArgs a) {
  static_assert(mixed_smem_bytes<Real, TS, SPLIT>() <= 160 * 1024, "LDS of one workgroup exceeds 160 KB");
  __shared__ __align__(16) char smem[mixed_smem_bytes<Real, TS, SPLIT>()];
  int sid = a.order ? a.order[blockIdx.x] : a.sid_base + (int)blockIdx.x;
  int part = 0;
  if constexpr (SPLIT) {
    if (a.split) {
      part = (int)((unsigned)sid >> 24);
      sid &= 0xffffff;
    }
  }
  if (sid < 0 || sid >= a.M) return;   // a caller-provided slot out of range: nothing to do
  const SolveDesc &D = a.desc[sid];
  switch (D.n * 8 + D.kpt) {
    case 3 * 8 + 1: sqp_solve<3, 1, Real, TS>(a, sid, part, smem); break;
    case 3 * 8 + 2: sqp_solve<3, 2, Real, TS>(a, sid, part, smem); break;
    case 6 * 8 + 1: sqp_solve<6, 1, Real, TS>(a, sid, part, smem); break;
    case 6 * 8 + 2: sqp_solve<6, 2, Real, TS>(a, sid, part, smem); break;
    case 7 * 8 + 1: sqp_solve<7, 1, Real, TS>(a, sid, part, smem); break;
    case 7 * 8 + 2: sqp_solve<7, 2, Real, TS>(a, sid, part, smem); break;
    case 6 * 8 + 4:
      if constexpr (!TS) sqp_solve<6, 4, Real, false, SPLIT>(a, sid, part, smem);
      else if constexpr (SPLIT && sizeof(Real) == 8) {
        if (task_split_ok(a, D, part)) sqp_solve_part<6, 1, true>(a, sid, part, smem);
      }
      break;
    case 7 * 8 + 4:
      if constexpr (!TS) sqp_solve<7, 4, Real, false, SPLIT>(a, sid, part, smem);
      else if constexpr (SPLIT && sizeof(Real) == 8) {
        if (task_split_ok(a, D, part)) sqp_solve_part<7, 1, true>(a, sid, part, smem);
      }
      break;
    default: break;  // the host only builds the shapes above
  }
}

}  // namespace gato
