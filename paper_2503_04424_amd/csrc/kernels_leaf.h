// Leaf kernels of the block-column factorisation (LEAF = 64 columns at a time).
//
// leaf_factor_kernel : in-place A = L D L^T of one <= 64 x 64 diagonal leaf
//                      (Sec. 2.2: "in-place ... decomposition" of the diagonal block,
//                      symmetric case: unit-lower L, diagonal D, no pivoting).
// leaf_factor_pivoted_kernel : the same with the pivot taken from the diagonal inside the
//                      leaf, P A P^T = L D L^T (Sec. 2.2: the symmetric form handles
//                      permutations; pivoting inside a block, none between blocks).
// leaf_lu_kernel     : a leaf of a general matrix, P A = L D U with unit-lower L, diagonal D
//                      and unit-upper U, the pivot of each column taken among the leaf's
//                      rows (Sec. 2.2, Eq. 1 and Alg. 1: M = P L U for generic matrices;
//                      pivoting inside a block, none between blocks).
// leaf_solve_kernel  : rows below the leaf, X = A_rows L^-T D^-1
//                      (Sec. 2.2: in-place triangular solve of the off-diagonal
//                      blocks; App. E.1 "solve lower triangular system"; the
//                      D^-1 is the LDL^T "diagonal scaling").  On request also
//                      W = X D into a second array, for the rows from `wfrom` on:
//                      the operand of the Schur updates with the scaling applied,
//                      rounded as the update kernels round l * d.
// leaf_solve_general_kernel : the same for both triangles of a general matrix in one
//                      launch (rows of the lower one against U^T, rows of the transposed
//                      upper one against L with the leaf's row order as column gather).
// transpose_strict_kernel : the entries above the diagonal of a general matrix into their
//                      transposed store, and back.
//
// The leaf kernels work on 16-column sub-blocks: the sequential part (elimination inside a
// 16 x 16 diagonal sub-block) runs on the vector ALUs with one matrix row per lane, everything
// else (the substitution against already solved sub-blocks with the inverse of the diagonal one,
// updates inside the leaf) is 16 x 16 x 16 products on the matrix cores.  The loops over the
// sub-blocks of a leaf that is factored are real loops around an unrolled elimination; those of
// a solve are unrolled, since its sub-blocks stay in registers.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "mfma.h"

namespace mdet {

constexpr int LEAF = 64;
constexpr int SUB = 16;               // sub-block order = MFMA tile order
constexpr int NSUB = LEAF / SUB;
constexpr int LEAF_PAD = LEAF + 1;    // LDS row stride of a leaf tile
constexpr int LEAF_TILE = LEAF * LEAF_PAD;

// Device-side status words shared by all kernels of one call.
struct DevFlags {
  unsigned long long first_bad;   // global index of the first zero / non-finite pivot; ~0 = none
  unsigned long long bad_kind;    // 1 = zero, 2 = non-finite
  unsigned long long odd_leaves;  // general matrices: leaves whose row order is an odd permutation
};

// Value of `v` in lane `src` (uniform lane index), delivered in scalar registers.
__device__ __forceinline__ double lane_value(double v, int src) {
  int lo = __builtin_amdgcn_readlane(__double2loint(v), src);
  int hi = __builtin_amdgcn_readlane(__double2hiint(v), src);
  return __hiloint2double(hi, lo);
}
__device__ __forceinline__ float lane_value(float v, int src) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), src));
}

// ---------------------------------------------------------------------------
// leaf factor
// ---------------------------------------------------------------------------
// 1/d to within a couple of ulp: hardware estimate refined by two Newton steps
// (the sequence an exact division expands to, minus its final correction and
// range scaling; pivots that would need scaling are far outside what a
// factorisation without pivoting can use anyway).
__device__ __forceinline__ double fast_rcp(double d) {
  double r = __builtin_amdgcn_rcp(d);
  r = fma(fma(-d, r, 1.0), r, r);
  r = fma(fma(-d, r, 1.0), r, r);
  return r;
}
__device__ __forceinline__ float fast_rcp(float d) {
  float r = __builtin_amdgcn_rcpf(d);
  r = fmaf(fmaf(-d, r, 1.0f), r, r);
  return r;
}

// w / d from the hardware estimate r of 1/d (relative error e < 2^-20): with e = 1 - d r,
// w/d = w r / (1 - e) = w r + w r (e + e^2 + ...); e^3 is below the last bit (fp32: e^2).
// quotient_tail is the bracket.  Within one ulp; three dependent operations behind the
// estimate.
__device__ __forceinline__ double rcp_estimate(double d) { return __builtin_amdgcn_rcp(d); }
__device__ __forceinline__ float rcp_estimate(float d) { return __builtin_amdgcn_rcpf(d); }
__device__ __forceinline__ double quotient_tail(double d, double r) {
  const double e = fma(-d, r, 1.0);
  return fma(e, e, e);
}
__device__ __forceinline__ float quotient_tail(float d, float r) { return fmaf(-d, r, 1.0f); }

// One step of Diag16 below: l = wm / pivot (from the estimate of 1 / pivot and the tail of its
// series), the updates of the columns behind J and of the inverse, the next pivot and the
// hardware's estimate of its reciprocal.  Written out because an operand that comes from
// another lane of the row (row_newbcast) is all but free only if it rides on the multiply-add,
// and the compiler makes a move of its own for each (a third more instructions).  A register
// must not be read that way within two instructions of being written by the vector ALU: the
// two instructions of the quotient cover what the compiler may put in front of the block, two
// updates (or waits) stand between the next pivot's column and its broadcast; and the estimate
// is not read by the instruction behind it.  (v_rcp_f64 itself with such an operand returns
// infinity on this chip.)
#define MDET_DPP(LANE) " row_newbcast:" LANE " row_mask:0xf bank_mask:0xf\n\t"
#define MDET_COL(Q) MDET_FMAC " %[d" Q "], %[w], %[nl]" MDET_DPP(Q)
#define MDET_COLS16 ""
#define MDET_COLS15 MDET_COL("15")
#define MDET_COLS14 MDET_COL("14") MDET_COLS15
#define MDET_COLS13 MDET_COL("13") MDET_COLS14
#define MDET_COLS12 MDET_COL("12") MDET_COLS13
#define MDET_COLS11 MDET_COL("11") MDET_COLS12
#define MDET_COLS10 MDET_COL("10") MDET_COLS11
#define MDET_COLS9 MDET_COL("9") MDET_COLS10
#define MDET_COLS8 MDET_COL("8") MDET_COLS9
#define MDET_COLS7 MDET_COL("7") MDET_COLS8
#define MDET_COLS6 MDET_COL("6") MDET_COLS7
#define MDET_COLS5 MDET_COL("5") MDET_COLS6
#define MDET_COLS4 MDET_COL("4") MDET_COLS5
#define MDET_OPS15 [d15] "+v"(d[15])
#define MDET_OPS14 [d14] "+v"(d[14]), MDET_OPS15
#define MDET_OPS13 [d13] "+v"(d[13]), MDET_OPS14
#define MDET_OPS12 [d12] "+v"(d[12]), MDET_OPS13
#define MDET_OPS11 [d11] "+v"(d[11]), MDET_OPS12
#define MDET_OPS10 [d10] "+v"(d[10]), MDET_OPS11
#define MDET_OPS9 [d9] "+v"(d[9]), MDET_OPS10
#define MDET_OPS8 [d8] "+v"(d[8]), MDET_OPS9
#define MDET_OPS7 [d7] "+v"(d[7]), MDET_OPS8
#define MDET_OPS6 [d6] "+v"(d[6]), MDET_OPS7
#define MDET_OPS5 [d5] "+v"(d[5]), MDET_OPS6
#define MDET_OPS4 [d4] "+v"(d[4]), MDET_OPS5
#define MDET_OPS3 [d3] "+v"(d[3]), MDET_OPS4
#define MDET_OPS2 [d2] "+v"(d[2]), MDET_OPS3
#define MDET_OPS1 [d1] "+v"(d[1]), MDET_OPS2
#define MDET_INV(S, J) MDET_FMAC " %[i" S "], %[i" S "], %[nl]" MDET_DPP(#J)
#define MDET_INVS1(J) MDET_INV("0", J)
#define MDET_INVS2(J) MDET_INVS1(J) MDET_INV("1", J)
#define MDET_INVS3(J) MDET_INVS2(J) MDET_INV("2", J)
#define MDET_INVS4(J) MDET_INVS3(J) MDET_INV("3", J)
#define MDET_WAIT1 "s_nop 0\n\t"
#define MDET_WAIT2 "s_nop 1\n\t"
// J, column J + 1, two more (or a wait), the rest, and the registers of the inverse in which
// row J has entries: acc_row(lane, s) <= J for some lane
#define MDET_STEP(J, J1, TWO, REST, OPS, INVS)                                                     \
  template <>                                                                                      \
  __device__ __forceinline__ void diag16_step<J>(MDET_T * d, MDET_T * inv, MDET_T w, MDET_T wm,    \
                                                 MDET_T tail, MDET_T & nl, MDET_T & next,          \
                                                 MDET_T & est) {                                   \
    MDET_T e = est;                                                                                \
    asm(MDET_MUL " %[p], -%[wm], %[es]\n\t" MDET_FMA " %[nl], %[p], %[t], %[p]\n\t"                \
            MDET_COL(J1) TWO MDET_MOV " %[p], %[d" J1 "]" MDET_DPP(J1) MDET_RCP " %[es], %[p]\n\t"  \
                REST INVS(J)                                                                       \
        : [nl] "=&v"(nl), [p] "=&v"(next), [es] "+v"(e), [i0] "+v"(inv[0]), [i1] "+v"(inv[1]),     \
          [i2] "+v"(inv[2]), [i3] "+v"(inv[3]), OPS                                                \
        : [w] "v"(w), [wm] "v"(wm), [t] "v"(tail));                                                \
    est = e;                                                                                       \
  }
template <int J, typename T>
__device__ __forceinline__ void diag16_step(T* d, T* inv, T w, T wm, T tail, T& nl, T& next, T& est);
#define MDET_T double
#define MDET_MUL "v_mul_f64"
#define MDET_FMA "v_fma_f64"
#define MDET_FMAC "v_fmac_f64_dpp"
#define MDET_MOV "v_mov_b64_dpp"
#define MDET_RCP "v_rcp_f64"
MDET_STEP(0, "1", MDET_COL("2") MDET_COL("3"), MDET_COLS4, MDET_OPS1, MDET_INVS1)
MDET_STEP(1, "2", MDET_COL("3") MDET_COL("4"), MDET_COLS5, MDET_OPS2, MDET_INVS1)
MDET_STEP(2, "3", MDET_COL("4") MDET_COL("5"), MDET_COLS6, MDET_OPS3, MDET_INVS1)
MDET_STEP(3, "4", MDET_COL("5") MDET_COL("6"), MDET_COLS7, MDET_OPS4, MDET_INVS1)
MDET_STEP(4, "5", MDET_COL("6") MDET_COL("7"), MDET_COLS8, MDET_OPS5, MDET_INVS2)
MDET_STEP(5, "6", MDET_COL("7") MDET_COL("8"), MDET_COLS9, MDET_OPS6, MDET_INVS2)
MDET_STEP(6, "7", MDET_COL("8") MDET_COL("9"), MDET_COLS10, MDET_OPS7, MDET_INVS2)
MDET_STEP(7, "8", MDET_COL("9") MDET_COL("10"), MDET_COLS11, MDET_OPS8, MDET_INVS2)
MDET_STEP(8, "9", MDET_COL("10") MDET_COL("11"), MDET_COLS12, MDET_OPS9, MDET_INVS3)
MDET_STEP(9, "10", MDET_COL("11") MDET_COL("12"), MDET_COLS13, MDET_OPS10, MDET_INVS3)
MDET_STEP(10, "11", MDET_COL("12") MDET_COL("13"), MDET_COLS14, MDET_OPS11, MDET_INVS3)
MDET_STEP(11, "12", MDET_COL("13") MDET_COL("14"), MDET_COLS15, MDET_OPS12, MDET_INVS3)
MDET_STEP(12, "13", MDET_COL("14") MDET_COL("15"), MDET_COLS16, MDET_OPS13, MDET_INVS4)
MDET_STEP(13, "14", MDET_COL("15") MDET_WAIT1, MDET_COLS16, MDET_OPS14, MDET_INVS4)
MDET_STEP(14, "15", MDET_WAIT2, MDET_COLS16, MDET_OPS15, MDET_INVS4)
#undef MDET_T
#undef MDET_MUL
#undef MDET_FMA
#undef MDET_FMAC
#undef MDET_MOV
#undef MDET_RCP
#define MDET_T float
#define MDET_MUL "v_mul_f32_e64"
#define MDET_FMA "v_fma_f32"
#define MDET_FMAC "v_fmac_f32_dpp"
#define MDET_MOV "v_mov_b32_dpp"
#define MDET_RCP "v_rcp_f32"
MDET_STEP(0, "1", MDET_COL("2") MDET_COL("3"), MDET_COLS4, MDET_OPS1, MDET_INVS1)
MDET_STEP(1, "2", MDET_COL("3") MDET_COL("4"), MDET_COLS5, MDET_OPS2, MDET_INVS2)
MDET_STEP(2, "3", MDET_COL("4") MDET_COL("5"), MDET_COLS6, MDET_OPS3, MDET_INVS3)
MDET_STEP(3, "4", MDET_COL("5") MDET_COL("6"), MDET_COLS7, MDET_OPS4, MDET_INVS4)
MDET_STEP(4, "5", MDET_COL("6") MDET_COL("7"), MDET_COLS8, MDET_OPS5, MDET_INVS4)
MDET_STEP(5, "6", MDET_COL("7") MDET_COL("8"), MDET_COLS9, MDET_OPS6, MDET_INVS4)
MDET_STEP(6, "7", MDET_COL("8") MDET_COL("9"), MDET_COLS10, MDET_OPS7, MDET_INVS4)
MDET_STEP(7, "8", MDET_COL("9") MDET_COL("10"), MDET_COLS11, MDET_OPS8, MDET_INVS4)
MDET_STEP(8, "9", MDET_COL("10") MDET_COL("11"), MDET_COLS12, MDET_OPS9, MDET_INVS4)
MDET_STEP(9, "10", MDET_COL("11") MDET_COL("12"), MDET_COLS13, MDET_OPS10, MDET_INVS4)
MDET_STEP(10, "11", MDET_COL("12") MDET_COL("13"), MDET_COLS14, MDET_OPS11, MDET_INVS4)
MDET_STEP(11, "12", MDET_COL("13") MDET_COL("14"), MDET_COLS15, MDET_OPS12, MDET_INVS4)
MDET_STEP(12, "13", MDET_COL("14") MDET_COL("15"), MDET_COLS16, MDET_OPS13, MDET_INVS4)
MDET_STEP(13, "14", MDET_COL("15") MDET_WAIT1, MDET_COLS16, MDET_OPS14, MDET_INVS4)
MDET_STEP(14, "15", MDET_WAIT2, MDET_COLS16, MDET_OPS15, MDET_INVS4)
#undef MDET_T
#undef MDET_MUL
#undef MDET_FMA
#undef MDET_FMAC
#undef MDET_MOV
#undef MDET_RCP
#undef MDET_STEP

// Elimination of a symmetric 16 x 16 block by one wavefront, right-looking, in registers.
// Every row of 16 lanes holds the whole block, row c in its lane c: d[q] = entry (c, q), the
// entries above the diagonal are not used.  Step J: l_c = d_cJ / pivot below the pivot, 0
// elsewhere; then d_cq -= l_c w_q for the columns q behind J, where w_q = d_qJ before its
// division comes from lane q of the same row of lanes as an operand of the multiply-add
// itself.  So no value crosses a row of lanes, and nothing goes through LDS or scalar
// registers from one pivot to the next.  The inverse of the unit-lower factor is carried
// along, its columns dealt out to the four rows of lanes: inv[s] of lane (c, g) is entry
// (c, k), k = acc_row(lane, s), the left-operand layout of the matrix instructions; row c of
// it receives -l_c times row J.
// A lone wavefront issues one instruction every four clocks (five with a lane operand), and
// that is what bounds this: about 24 a step.  Measured: 1970 clocks a block in fp64, 1690 in
// fp32.  One copy of the block spread over the four rows of lanes does a quarter of the
// updates, but bringing the pivot row to all of them costs eight instructions a step with
// their wait states (3480 clocks); with the exchange as separate moves it is 2590.
// stored: where entry (c, g) of L and D goes in memory, for c < rows; written four columns at
// a time.  On return mypiv is pivot c.
// THROUGH: as in leaf_factor_body.
template <bool THROUGH, typename T>
__device__ __forceinline__ void leaf_store(T* p, T v) {
  if constexpr (THROUGH) __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  else *p = v;
}
template <typename T, bool THROUGH = false>
struct Diag16 {
  using X = Mfma<T>;
  T d[SUB];
  T inv[4];
  T mypiv;
  T nl4[4];

  template <int J>
  __device__ __forceinline__ void steps(const int c, const int g, T piv, T est, T* stored, const int rows) {
    const T w = d[J];
    mypiv = c > J - 1 ? w : mypiv;                // lane c keeps the last: its own
    if constexpr (J + 1 < SUB) {
      T next;
      diag16_step<J>(d, inv, w, c > J ? w : T(0), quotient_tail(piv, est), nl4[J & 3], next, est);
      if constexpr ((J & 3) == 3) store<J / 4>(c, g, stored, rows);
      steps<J + 1>(c, g, next, est, stored, rows);
    } else {
      nl4[J & 3] = T(0);
      store<J / 4>(c, g, stored, rows);
    }
  }
  template <int Q>
  __device__ __forceinline__ void store(const int c, const int g, T* stored, const int rows) {
    const T lo = (g & 1) ? nl4[1] : nl4[0], hi = (g & 1) ? nl4[3] : nl4[2];
    const int k = 4 * Q + g;
    const T v = c == k ? mypiv : -((g & 2) ? hi : lo);
    if (k <= c && c < rows) leaf_store<THROUGH>(stored + 4 * Q, v);
  }
  __device__ __forceinline__ void eliminate(const int lane, T* stored, const int rows) {
    const int c = lane & 15, g = lane >> 4;
#pragma unroll
    for (int s = 0; s < 4; ++s) inv[s] = X::acc_row(lane, s) == c ? T(1) : T(0);
    mypiv = T(0);
    T piv = lane_value(d[0], 0);                // the same in every row of lanes
    steps<0>(c, g, piv, rcp_estimate(piv), stored, rows);
  }
};

// v -= sum_k h[k] w_k for the first 4, 8, 12 or 16 k, w_k in lane k of each row of 16 lanes (the wait
// covers the instruction that made w, see MDET_STEP)
#define MDET_APPLY_TERM(K, H) MDET_FMAC " %0, -%1, %" H " row_newbcast:" K " row_mask:0xf bank_mask:0xf\n\t"
#define MDET_APPLY_TERMS4 MDET_APPLY_TERM("0", "2") MDET_APPLY_TERM("1", "3") MDET_APPLY_TERM("2", "4") MDET_APPLY_TERM("3", "5")
#define MDET_APPLY_TERMS8 \
  MDET_APPLY_TERMS4 MDET_APPLY_TERM("4", "6") MDET_APPLY_TERM("5", "7") MDET_APPLY_TERM("6", "8") MDET_APPLY_TERM("7", "9")
#define MDET_APPLY_TERMS12 \
  MDET_APPLY_TERMS8 MDET_APPLY_TERM("8", "10") MDET_APPLY_TERM("9", "11") MDET_APPLY_TERM("10", "12") MDET_APPLY_TERM("11", "13")
#define MDET_APPLY_TERMS16 \
  MDET_APPLY_TERMS12 MDET_APPLY_TERM("12", "14") MDET_APPLY_TERM("13", "15") MDET_APPLY_TERM("14", "16") MDET_APPLY_TERM("15", "17")
#define MDET_H4 "v"(h[0]), "v"(h[1]), "v"(h[2]), "v"(h[3])
#define MDET_H8 MDET_H4, "v"(h[4]), "v"(h[5]), "v"(h[6]), "v"(h[7])
#define MDET_H12 MDET_H8, "v"(h[8]), "v"(h[9]), "v"(h[10]), "v"(h[11])
#define MDET_H16 MDET_H12, "v"(h[12]), "v"(h[13]), "v"(h[14]), "v"(h[15])
#define MDET_APPLY(TYPE, N) asm("s_nop 1\n\t" MDET_APPLY_TERMS##N : "+&v"(v) : "v"(w), MDET_H##N)
#define MDET_APPLY_ALL(TYPE)                                                                 \
  template <int N>                                                                           \
  __device__ __forceinline__ void apply_terms(TYPE& v, const TYPE (&h)[16], TYPE w) {        \
    static_assert(N == 4 || N == 8 || N == 12 || N == 16, "terms in fours");                 \
    if constexpr (N == 4) MDET_APPLY(TYPE, 4);                                               \
    else if constexpr (N == 8) MDET_APPLY(TYPE, 8);                                          \
    else if constexpr (N == 12) MDET_APPLY(TYPE, 12);                                        \
    else MDET_APPLY(TYPE, 16);                                                               \
  }
#define MDET_FMAC "v_fmac_f64_dpp"
MDET_APPLY_ALL(double)
#undef MDET_FMAC
#define MDET_FMAC "v_fmac_f32_dpp"
MDET_APPLY_ALL(float)
#undef MDET_FMAC
#undef MDET_APPLY_ALL
#undef MDET_APPLY_TERM
#undef MDET_APPLY
#undef MDET_H16
#undef MDET_H12
#undef MDET_H8
#undef MDET_H4
#undef MDET_APPLY_TERMS16
#undef MDET_APPLY_TERMS12
#undef MDET_APPLY_TERMS8
#undef MDET_APPLY_TERMS4
// The first j terms (the registers of the others hold zeros): j is known where a loop is unrolled.  One sum, which
// starts from the entry and takes its terms in their order: even and odd terms apart, which would wait less for
// each other, gain nothing (a leaf 1 % slower, in fp32 6 %) and round to the size of the terms and not of what is left of the entry.
template <typename T>
__device__ __forceinline__ void apply_first(T& v, const T (&h)[16], T w, const int j) {
  if (j > 12) apply_terms<16>(v, h, w);
  else if (j > 8) apply_terms<12>(v, h, w);
  else if (j > 4) apply_terms<8>(v, h, w);
  else if (j > 0) apply_terms<4>(v, h, w);
}

// Inverse of a unit-lower 16 x 16 block -> linv (16 x 16, row-major), by one wavefront: nl[k]
// of lane (c, g) is minus entry (c, k) of the block below the diagonal (c > k), 0 elsewhere.
// As in Diag16, row c in lane c, the columns dealt out to the four rows of lanes: step k adds
// nl_ck times row k, read from lane k by the multiply-add itself.  64 instructions and no
// memory in between; substituting column by column with the block's entries as LDS broadcasts
// took 3000 clocks, ten times as long.  (Four registers in turn, so that none is read from
// another lane within two instructions of being written.)
#define MDET_INV_ROW(K, N)                                                                           \
  MDET_FMAC " %0, %0, %" N MDET_DPP(K) MDET_FMAC " %1, %1, %" N MDET_DPP(K)                          \
      MDET_FMAC " %2, %2, %" N MDET_DPP(K) MDET_FMAC " %3, %3, %" N MDET_DPP(K)
#define MDET_INVERT16(TYPE)                                                                          \
  __device__ __forceinline__ void invert16_rows(TYPE (&x)[4], const TYPE (&nl)[SUB]) {               \
    asm("s_nop 1\n\t" MDET_INV_ROW("0", "4") MDET_INV_ROW("1", "5") MDET_INV_ROW("2", "6")           \
            MDET_INV_ROW("3", "7") MDET_INV_ROW("4", "8") MDET_INV_ROW("5", "9")                     \
                MDET_INV_ROW("6", "10") MDET_INV_ROW("7", "11") MDET_INV_ROW("8", "12")              \
                    MDET_INV_ROW("9", "13") MDET_INV_ROW("10", "14") MDET_INV_ROW("11", "15")        \
                        MDET_INV_ROW("12", "16") MDET_INV_ROW("13", "17") MDET_INV_ROW("14", "18")   \
        : "+v"(x[0]), "+v"(x[1]), "+v"(x[2]), "+v"(x[3])                                             \
        : "v"(nl[0]), "v"(nl[1]), "v"(nl[2]), "v"(nl[3]), "v"(nl[4]), "v"(nl[5]), "v"(nl[6]),        \
          "v"(nl[7]), "v"(nl[8]), "v"(nl[9]), "v"(nl[10]), "v"(nl[11]), "v"(nl[12]), "v"(nl[13]),    \
          "v"(nl[14]));                                                                              \
  }
#define MDET_FMAC "v_fmac_f64_dpp"
MDET_INVERT16(double)
#undef MDET_FMAC
#define MDET_FMAC "v_fmac_f32_dpp"
MDET_INVERT16(float)
#undef MDET_FMAC
#undef MDET_INVERT16
#undef MDET_INV_ROW
template <typename T>
__device__ __forceinline__ void invert16(const T (&nl)[SUB], T* __restrict__ linv, const int lane) {
  const int c = lane & 15;
  T x[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) x[s] = Mfma<T>::acc_row(lane, s) == c ? T(1) : T(0);
  invert16_rows(x, nl);
#pragma unroll
  for (int s = 0; s < 4; ++s) linv[c * SUB + Mfma<T>::acc_row(lane, s)] = x[s];
}
// The same for diagonal sub-block b of the unit-lower leaf in `tile` -> its place in linv.
template <typename T>
__device__ __forceinline__ void leaf_invert_sub(const T* tile, T* __restrict__ linv, const int b,
                                                const int lane) {
  const int c = lane & 15;
  const T* row = tile + (b * SUB + c) * LEAF_PAD + b * SUB;
  T nl[SUB];
#pragma unroll
  for (int k = 0; k < SUB; ++k) nl[k] = row[k];
#pragma unroll
  for (int k = 0; k < SUB; ++k) nl[k] = c > k ? -nl[k] : T(0);
  invert16<T>(nl, linv + b * SUB * SUB, lane);
}

// Four wavefronts factor one leaf held in LDS, on 16 x 16 sub-blocks.  Sub-block (i, j) of the
// upper half, i <= j, stands for the transpose of the stored sub-block (j, i); in accumulator
// layout a lane's four registers of X_ij are at the same time X_ij as a right operand and its
// transpose as a left operand of the matrix instructions (both index the inner dimension by
// acc_row), so the products below need no change of layout:
//     U_bj = L_bb^-1 S_bj,     L_jb^T = D_b^-1 U_bj,     S_ij -= L_ib U_bj.
// Wavefront 0 has the chain of dependent steps to itself: eliminate diagonal block b with the
// inverse of its factor, hand the inverse and the pivots to the others, form U_b,b+1 and the
// next diagonal block from it, and go on, while wavefronts 1 to 3 do the products off that
// chain (they form the U they need themselves) and write L and the pivots to memory.
// Measured, one leaf with its load from memory and its launch: 8.2 us in fp64, 6.9 in fp32;
// with one panel of 16 columns and the rows below it eliminated through LDS at a time, and
// the rank-16 updates of the leaf between barriers, 10.7 and 9.5.  What is left per diagonal
// block: 1970 clocks of elimination, about 1000 for the two products and the change of layout
// in front of it, 400 for the hand-over.
constexpr int FACTOR_THREADS = 256;

// LDS the factorisation needs, in elements: the leaf, the inverses of two diagonal blocks in
// turn, the pivots and reciprocals of all, and a block changing layout.
constexpr int FACTOR_LDS_ELEMS = LEAF_TILE + 2 * SUB * SUB + 2 * LEAF + SUB * SUB;

// The work of all FACTOR_THREADS threads of one workgroup; `lds` points at
// FACTOR_LDS_ELEMS elements of shared memory nobody else uses.  The update
// kernels call it too: the workgroup that has just reduced the top-left 64 x 64
// block of its launch factors that block straight away, which takes one kernel
// (and its launch-to-launch latency) off the chain of dependent launches.
//
// With IN_LDS the caller has put the leaf into `lds` already, entry by entry with
// leaf_tile_put and a barrier after the last one (an update kernel hands over its
// accumulators: writing the block to memory and reading it back would cost a memory
// round trip on the chain of dependent launches); A is then only written.
template <typename T>
__device__ __forceinline__ void leaf_tile_put(T* __restrict__ lds, int row, int col, int w, T v) {
  if (row < LEAF && col < LEAF)
    lds[row * LEAF_PAD + col] = (row < w && col < w) ? v : (row == col ? T(1) : T(0));
}

//
// spd != 0: the positive-definite form.  The leaf is still factored as L D L^T, but
// every pivot must be positive (the first that is not is reported with kind 4) and
// dinv receives d^(-1/2) instead of 1/d: the rows below the leaf, solved with that
// scaling, are then rows of the Cholesky factor L D^(1/2), and the updates that use
// them need no pivots.
//
// THROUGH: what is stored is for workgroups of the same launch, on other chiplets too: stores at
// device scope, past this chiplet's L2 cache.  They form the inverses themselves (linv is not used).
// Wavefronts beyond the fourth only keep the barriers company, and the other three may come to the
// first of them late: only sub-block (0, 0) has to be in LDS, put there by wavefront 0 itself, when
// that begins.  Behind the first barrier *mid becomes mid_value.
template <typename T, bool IN_LDS = false, bool THROUGH = false>
__device__ __forceinline__ void leaf_factor_body(
    T* __restrict__ A, int64_t ld, int w, T* __restrict__ dvec, T* __restrict__ dinv,
    T* __restrict__ linv, long long pivot0, DevFlags* flags, T* __restrict__ lds, int spd = 0,
    unsigned* mid = nullptr, unsigned mid_value = 0u) {
  using X = Mfma<T>;
  using acc_t = typename X::acc_t;
  T* tile = lds;
  // The elimination is one long chain of dependent instructions; beside a
  // workgroup of the trailing update on the same SIMDs it would otherwise get an
  // issue slot only now and then.
  __builtin_amdgcn_s_setprio(3);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // the same in all lanes: scalar branches
  const int l16 = lane & 15, g = lane >> 4;
  if constexpr (!IN_LDS) {
    // 64 x 64 tile, 16 entries per thread, all requests in flight together
    T v[LEAF * LEAF / FACTOR_THREADS];
#pragma unroll
    for (int q = 0; q < LEAF * LEAF / FACTOR_THREADS; ++q) {
      const int e = q * FACTOR_THREADS + tid, r = e >> 6, c = e & 63;
      v[q] = (r < w && c < w) ? A[(int64_t)r * ld + c] : (r == c ? T(1) : T(0));
    }
#pragma unroll
    for (int q = 0; q < LEAF * LEAF / FACTOR_THREADS; ++q) {
      const int e = q * FACTOR_THREADS + tid, r = e >> 6, c = e & 63;
      tile[r * LEAF_PAD + c] = v[q];
    }
    __syncthreads();
  }

  T* inv_of = tile + LEAF_TILE;                  // [2][4][64]
  T* piv_of = inv_of + 2 * SUB * SUB;            // [64]
  T* rcp_of = piv_of + LEAF;                     // [64]
  T* turn = rcp_of + LEAF;                       // [16][16]
  // place of entry s of this lane's share of sub-block (i, j), i <= j
  auto at = [&](const int i, const int j, const int s) -> T& {
    return tile[(j * SUB + l16) * LEAF_PAD + i * SUB + X::acc_row(lane, s)];
  };
  // U_pj = L_pp^-1 S_pj and L_jp^T
  auto solve_sub = [&](const int p, const int j, const T (&inv)[4], const T (&rk)[4], acc_t& u, T (&l)[4]) {
    T x[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) x[s] = at(p, j, s);
    u = acc_t{0, 0, 0, 0};
#pragma unroll
    for (int s = 0; s < 4; ++s) u = X::mfma(inv[s], x[s], u);
#pragma unroll
    for (int s = 0; s < 4; ++s) l[s] = u[s] * rk[s];
  };
  auto product = [&](acc_t c, const T (&l)[4], const acc_t& u) {
#pragma unroll
    for (int s = 0; s < 4; ++s) c = X::mfma(-l[s], u[s], c);
    return c;
  };
  auto load_sub = [&](const int i, const int j) {
    acc_t c;
#pragma unroll
    for (int s = 0; s < 4; ++s) c[s] = at(i, j, s);
    return c;
  };
  // L of sub-block (j, p) to memory
  auto store_l = [&](const int j, const int p, const T (&l)[4]) {
    const int r = j * SUB + l16;
#pragma unroll
    for (int s = 0; s < 4; ++s)
      if (r < w) leaf_store<THROUGH>(A + (int64_t)r * ld + p * SUB + X::acc_row(lane, s), l[s]);
  };
  // the pivots of diagonal block p to memory
  auto store_pivots = [&](const int p) {
    const int i = p * SUB + l16;
    if (g == 0 && i < w) {
      const T d = piv_of[i];
      leaf_store<THROUGH>(dvec + i, d);
      leaf_store<THROUGH>(dinv + i, T(spd != 0 ? T(1) / sqrt(d) : rcp_of[i]));
    }
  };

  Diag16<T, THROUGH> dg;
#pragma unroll 1
  for (int b = 0; b < NSUB; ++b) {
    const int p = b - 1;                          // the diagonal block done last
    T inv[4], rk[4];
    if (wave == 0) {
      if (b == 0) {
#pragma unroll
        for (int q = 0; q < SUB; ++q) dg.d[q] = tile[l16 * LEAF_PAD + q];
      } else {
        acc_t u, c = load_sub(b, b);
        T l[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) rk[s] = rcp_of[p * SUB + X::acc_row(lane, s)];
        solve_sub(p, b, dg.inv, rk, u, l);
        c = product(c, l, u);
        // (a wavefront's LDS operations complete in the order they were issued)
#pragma unroll
        for (int s = 0; s < 4; ++s) turn[X::acc_row(lane, s) * SUB + l16] = c[s];
#pragma unroll
        for (int q = 0; q < SUB; ++q) dg.d[q] = turn[q * SUB + l16];
      }
      dg.eliminate(lane, A + (int64_t)(b * SUB + l16) * ld + b * SUB + g, w - b * SUB);
#pragma unroll
      for (int s = 0; s < 4; ++s) inv_of[((b & 1) * 4 + s) * 64 + lane] = dg.inv[s];
      piv_of[b * SUB + l16] = dg.mypiv;
      rcp_of[b * SUB + l16] = fast_rcp(dg.mypiv);
      if constexpr (!THROUGH) {
#pragma unroll
        for (int s = 0; s < 4; ++s) linv[(b * SUB + l16) * SUB + X::acc_row(lane, s)] = dg.inv[s];
      }
    } else if (b > 0 && (!THROUGH || wave < 4)) {
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        inv[s] = inv_of[((p & 1) * 4 + s) * 64 + lane];
        rk[s] = rcp_of[p * SUB + X::acc_row(lane, s)];
      }
      // sub-blocks, one wavefront's after the other:
      // b = 1: (1,2) (2,2) | (1,3) (3,3) | (2,3);  b = 2: (2,3) | (3,3);  b = 3: none
      const int j = b == 1 && wave == 1 ? 2 : 3;
      const int i = b == 1 && wave < 3 ? 1 : 2;
      const bool cross = b == 1 || (b == 2 && wave == 1);
      const bool self = (b == 1 && wave < 3) || (b == 2 && wave == 2);
      const bool lonely = b == 3 && wave == 1;    // nobody else writes L_32
      acc_t u;
      T l[4];
      if (cross || self || lonely) solve_sub(p, j, inv, rk, u, l);
      if (cross) {
        acc_t ui;
        T li[4];
        solve_sub(p, i, inv, rk, ui, li);
        const acc_t c = product(load_sub(i, j), li, u);
#pragma unroll
        for (int s = 0; s < 4; ++s) at(i, j, s) = c[s];
        if (wave == 1) store_l(i, p, li);         // L_10, L_21
      }
      if (self) {
        const acc_t c = product(load_sub(j, j), l, u);
#pragma unroll
        for (int s = 0; s < 4; ++s) at(j, j, s) = c[s];
      }
      if (self || lonely) store_l(j, p, l);       // L_20, L_30 | L_31 | L_32
      if (wave == 3) store_pivots(p);
    }
    if (b + 1 < NSUB) __syncthreads();
    if constexpr (THROUGH) {
      if (b == 0 && tid == 64) __hip_atomic_store(mid, mid_value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
  // the last pivots, and the first zero / non-finite one of all through the flags (wavefront 0
  // reads LDS entries of its own: no barrier)
  if (wave == 0) {
    store_pivots(NSUB - 1);
    const T myd = piv_of[lane];
    const bool zero = myd == T(0);
    const bool finite = fabs((double)myd) <= 1.7976931348623157e308;
    const unsigned long long mask = __ballot(lane < w && (zero || !finite || (spd != 0 && myd < T(0))));
    if (mask != 0ull && lane == __ffsll((long long)mask) - 1) {
      const unsigned long long idx = (unsigned long long)(pivot0 + lane);
      const unsigned long long old = atomicMin(&flags->first_bad, idx);
      if (idx <= old) atomicExch(&flags->bad_kind, zero ? 1ull : (!finite ? 2ull : 4ull));
    }
  }
  __builtin_amdgcn_s_setprio(0);
}

template <typename T>
__global__ __launch_bounds__(FACTOR_THREADS) void leaf_factor_kernel(
    T* __restrict__ A, int64_t ld, int w, T* __restrict__ dvec, T* __restrict__ dinv,
    T* __restrict__ linv, long long pivot0, DevFlags* flags, int spd) {
  __shared__ T lds[FACTOR_LDS_ELEMS];
  leaf_factor_body<T>(A, ld, w, dvec, dinv, linv, pivot0, flags, lds, spd);
}

// ---------------------------------------------------------------------------
// leaf factor with pivoting
// ---------------------------------------------------------------------------
// Maximum of x over the 64 lanes, delivered in a scalar register: four exchanges inside each row of
// 16 lanes on the data-parallel-primitive path, then the four rows' values through scalar registers (two
// more exchanges, with the copies that the compiler makes for them, take 25 clocks longer).  Must be reached by
// all 64 lanes.
__device__ __forceinline__ unsigned wave_max_u32(unsigned x) {
  int m = (int)x;
  auto take = [&](int other) { m = (int)max((unsigned)m, (unsigned)other); };
  take(__builtin_amdgcn_update_dpp(0, m, 0xB1, 0xF, 0xF, false));    // lanes 1 0 3 2 of each four
  take(__builtin_amdgcn_update_dpp(0, m, 0x4E, 0xF, 0xF, false));    // lanes 2 3 0 1
  take(__builtin_amdgcn_update_dpp(0, m, 0x141, 0xF, 0xF, false));   // mirror inside each eight
  take(__builtin_amdgcn_update_dpp(0, m, 0x140, 0xF, 0xF, false));   // mirror inside each sixteen
  const unsigned r0 = (unsigned)__builtin_amdgcn_readlane(m, 0), r1 = (unsigned)__builtin_amdgcn_readlane(m, 16);
  const unsigned r2 = (unsigned)__builtin_amdgcn_readlane(m, 32), r3 = (unsigned)__builtin_amdgcn_readlane(m, 48);
  return max(max(r0, r1), max(r2, r3));
}

// LDS that wavefronts exchange without a barrier: accesses stay in the order they are written
// in, and in LDS instructions (through a generic pointer they would be memory instructions,
// each waited for).
template <typename T>
using lds_volatile = volatile __attribute__((address_space(3))) T;

// The pivot rule: the lane of `cand` whose v is largest in magnitude, the lowest
// one on ties.  Magnitudes of IEEE numbers order like their bit patterns without the sign; a
// NaN is above all others, so that it is taken and reported.  Must be reached by all 64 lanes.  (`cand`
// empty: the last lane.)
__device__ __forceinline__ int pick_lane(double v, unsigned long long cand) {
  const bool mine = __builtin_amdgcn_inverse_ballot_w64(cand);
  const unsigned hi = (unsigned)__double2hiint(v) & 0x7fffffffu;
  const unsigned top_hi = wave_max_u32(mine ? hi : 0u);
  unsigned long long hit = __builtin_amdgcn_ballot_w64(hi == top_hi) & cand;
  // the upper words (exponent, 20 bits of the fraction) nearly always decide
  if (__builtin_expect((hit & (hit - 1ull)) != 0ull, 0)) {
    const bool level = __builtin_amdgcn_inverse_ballot_w64(hit);
    const unsigned lo = (unsigned)__double2loint(v);
    const unsigned top_lo = wave_max_u32(level ? lo : 0u);
    hit &= __builtin_amdgcn_ballot_w64(lo == top_lo);
  }
  return __builtin_ctzll(hit | 1ull << 63);
}
__device__ __forceinline__ int pick_lane(float v, unsigned long long cand) {
  const bool mine = __builtin_amdgcn_inverse_ballot_w64(cand);
  const unsigned key = __float_as_uint(v) & 0x7fffffffu;
  const unsigned top = wave_max_u32(mine ? key : 0u);
  return __builtin_ctzll(__builtin_amdgcn_ballot_w64(key == top) & cand | 1ull << 63);
}

// One leaf, P A P^T = L D L^T with P chosen inside the leaf: at every step the largest
// remaining diagonal entry of the Schur complement is the pivot.  Nothing is swapped while the
// elimination runs; lane c stands for row and column c.  The leaf is a full symmetric matrix
// in LDS, brought up to date with 16 steps at a time on the matrix cores by all wavefronts;
// the steps themselves are wavefront 0's.  Step j, pivot p: row p is read from LDS, v_c; the
// steps of the same 16 are applied to it, v_c -= l_kc (l_kp d_k), with l_kc in registers and the
// bracket from lane k of the row of lanes; l_c = v_c / d for the rows still to come; the running diagonal, in registers,
// receives -l_c v_c.  So a row that has been taken keeps its pivot there, and the next
// pivot can be looked for at once.  The multipliers are kept by step and input row, and put
// into the order in which the rows were taken when they are written to memory.
// Outputs as leaf_factor_kernel (L and D in pivot order into A, pivots, reciprocals,
// inverses of the diagonal sub-blocks of L), and perm[j] = pivot0 + (row taken at step j).
// Bound by the chain of one step (430 clocks: search 230, row from LDS 100, its terms so far, quotient);
// the three products between cost 2500 clocks each.  Measured, fp64, inside panel_flow_kernel: 15.5 us a leaf,
// 23.1 from one leaf to the next (with all 16 terms a step whatever their number, and the tile left of the leaf stored and
// the multipliers' places cleared in front of it, 26.4; n = 4096 1.69 -> 1.60 ms).
// IN_LDS, THROUGH: as for leaf_factor_body; `lds` has PIVOT_LDS_ELEMS elements, of which with IN_LDS
// the first LEAF_TILE hold the leaf, both triangles, row stride LEAF_PAD.  With THROUGH the other
// wavefronts do what `beside` says during the first 16 steps, and when that is in memory *mid becomes
// mid_value.  cleared: the multipliers' places (LEAF_TILE behind the leaf) are zero already.
constexpr int PIVOT_WAVES = 8;
constexpr int PIVOT_LDS_ELEMS = 2 * LEAF_TILE + 2 * LEAF;
struct LeafBeside {
  __device__ __forceinline__ void operator()() const {}
};
template <typename T, bool IN_LDS = false, bool THROUGH = false, typename Beside = LeafBeside>
__device__ __forceinline__ void leaf_factor_pivoted_body(
    T* __restrict__ A, int64_t ld, int w, T* __restrict__ dvec, T* __restrict__ dinv,
    T* __restrict__ linv, int* __restrict__ perm, long long pivot0, DevFlags* flags, T* __restrict__ lds,
    unsigned* mid = nullptr, unsigned mid_value = 0u, const Beside& beside = Beside{}, const bool cleared = false) {
  using X = Mfma<T>;
  using acc_t = typename X::acc_t;
  constexpr int NW = PIVOT_WAVES;
  T* const S = lds;
  T* const mult = S + LEAF_TILE;  // multipliers: by step, input row (0 for rows taken before)
  T* const dl = mult + LEAF_TILE; // pivots in the order taken
  int* const row_of = reinterpret_cast<int*>(dl + LEAF);   // row taken at a step
  __builtin_amdgcn_s_setprio(3);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15;
  if constexpr (!IN_LDS) {
    // one row a load; the padding of a narrow leaf is the identity
    T v[LEAF / NW];
#pragma unroll
    for (int k = 0; k < LEAF / NW; ++k) {
      const int r = NW * k + wave;
      v[k] = (r < w && lane <= r) ? A[(int64_t)r * ld + lane] : (r == lane ? T(1) : T(0));
    }
#pragma unroll
    for (int k = 0; k < LEAF / NW; ++k) {
      const int r = NW * k + wave;
      if (lane <= r) {
        S[r * LEAF_PAD + lane] = v[k];
        S[lane * LEAF_PAD + r] = v[k];
      }
    }
  }
  if (!cleared)
    for (int e = tid; e < LEAF_TILE; e += 64 * NW) mult[e] = T(0);
  __syncthreads();
  T diag = S[lane * LEAF_PAD + lane];
  // rows still to be taken: those of the leaf, and when there are none left (w < 64) those of the padding,
  // whose pivots are their own ones and eliminate nothing
  unsigned long long left = w < LEAF ? (1ull << w) - 1ull : ~0ull;
  const unsigned long long padding = ~left;
#pragma unroll 1
  for (int m = 0; m < NSUB; ++m) {
    if (wave == 0) {
      // dm, pm: pivot and row of step k of the 16 in lane k of each row of lanes
      T l[SUB], dm = T(0);
      int pm = 0, mine = l16;
      asm volatile("" : "+v"(mine));         // compared here, not kept as 16 masks in scalar registers
#pragma unroll
      for (int k = 0; k < SUB; ++k) l[k] = T(0);
      const T* const terms = mult + (m * SUB + l16) * LEAF_PAD;
      T* const to = mult + m * SUB * LEAF_PAD + lane;
#pragma unroll
      for (int j = 0; j < SUB; ++j) {
        left = left != 0ull ? left : padding;
        const int p = pick_lane(diag, left);
        T v = S[p * LEAF_PAD + lane];
        const T lp = terms[p];
        const T d = lane_value(diag, p);
        const T est = rcp_estimate(d);
        const T tail = quotient_tail(d, est);
        left &= ~(1ull << p);
        apply_first(v, l, lp * dm, j);
        dm = mine == j ? d : dm;
        const T q = v * est;
        l[j] = __builtin_amdgcn_inverse_ballot_w64(left) ? fma(q, tail, q) : T(0);
        diag = fma(-l[j], v, diag);
        to[j * LEAF_PAD] = l[j];
        pm = mine == j ? p : pm;
      }
      dl[m * SUB + l16] = dm;                // (the four rows of lanes: the same values)
      row_of[m * SUB + l16] = pm;
    } else if (THROUGH && m == 0) {
      beside();
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
    __syncthreads();
    if constexpr (THROUGH) {
      if (m == 0 && tid == 64) __hip_atomic_store(mid, mid_value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (m + 1 < NSUB) {
      // S -= L D L^T of these 16 steps, all of it: row p is wanted, whatever p.  Two of the
      // 16 sub-blocks a wavefront, side by side
      static_assert(2 * PIVOT_WAVES == NSUB * NSUB, "two sub-blocks a wavefront");
      const int R = (wave >> 1) * SUB, C = (wave & 1) * 2 * SUB;
      acc_t acc[2];
      T aop[4], bop[2][4];
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const int k = m * SUB + X::acc_row(lane, s);
        aop[s] = -(mult[k * LEAF_PAD + R + l16] * dl[k]);
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          bop[t][s] = mult[k * LEAF_PAD + C + t * SUB + l16];
          acc[t][s] = S[(R + X::acc_row(lane, s)) * LEAF_PAD + C + t * SUB + l16];
        }
      }
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int t = 0; t < 2; ++t) acc[t] = X::mfma(aop[s], bop[t][s], acc[t]);
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int t = 0; t < 2; ++t) S[(R + X::acc_row(lane, s)) * LEAF_PAD + C + t * SUB + l16] = acc[t][s];
      __syncthreads();
    }
  }
  // L and D in the order in which the rows were taken
  {
    T v[LEAF / NW];
#pragma unroll
    for (int k = 0; k < LEAF / NW; ++k) v[k] = mult[lane * LEAF_PAD + row_of[NW * k + wave]];
    const T myd = dl[lane];
#pragma unroll
    for (int k = 0; k < LEAF / NW; ++k) {
      const int r = NW * k + wave;
      if (r < w && lane <= r) leaf_store<THROUGH>(A + (int64_t)r * ld + lane, lane == r ? myd : v[k]);
    }
  }
  if (!THROUGH && wave < NSUB) {
    const int c = row_of[wave * SUB + l16];
    T nl[SUB];
#pragma unroll
    for (int k = 0; k < SUB; ++k) nl[k] = mult[(wave * SUB + k) * LEAF_PAD + c];
#pragma unroll
    for (int k = 0; k < SUB; ++k) nl[k] = l16 > k ? -nl[k] : T(0);
    invert16<T>(nl, linv + wave * SUB * SUB, lane);
  }
  if (wave == NW - 1) {
    const T myd = dl[lane];
    const bool zero = myd == T(0);
    const bool finite = fabs((double)myd) <= 1.7976931348623157e308;
    const bool bad = lane < w && (zero || !finite);
    if (lane < w) {
      leaf_store<THROUGH>(dvec + lane, myd);
      leaf_store<THROUGH>(dinv + lane, fast_rcp(myd));
      leaf_store<THROUGH>(perm + lane, (int)pivot0 + row_of[lane]);
    }
    const unsigned long long mask = __ballot(bad);
    if (mask != 0ull) {
      const int first = __ffsll((long long)mask) - 1;
      if (lane == first) {
        unsigned long long idx = (unsigned long long)(pivot0 + first);
        unsigned long long old = atomicMin(&flags->first_bad, idx);
        if (idx <= old) atomicExch(&flags->bad_kind, zero ? 1ull : 2ull);
      }
    }
  }
  __builtin_amdgcn_s_setprio(0);
}
template <typename T>
__global__ __launch_bounds__(64 * PIVOT_WAVES) void leaf_factor_pivoted_kernel(
    T* __restrict__ A, int64_t ld, int w, T* __restrict__ dvec, T* __restrict__ dinv,
    T* __restrict__ linv, int* __restrict__ perm, long long pivot0, DevFlags* flags) {
  __shared__ T lds[PIVOT_LDS_ELEMS];
  leaf_factor_pivoted_body<T>(A, ld, w, dvec, dinv, linv, perm, pivot0, flags, lds);
}

// ---------------------------------------------------------------------------
// leaf factor, general matrix
// ---------------------------------------------------------------------------
// The library keeps a general matrix as two lower-triangular arrays of the same shape:
// Pl holds the entries on and below the diagonal, Qu the entries above it, transposed
// (Qu[i][j] = M[j][i], i > j), so that both halves of every block row and column are read
// along rows, as the update and solve kernels want their operands.  This kernel factors
// one <= 64 x 64 diagonal leaf, given as its two halves: P A = L D U by Gaussian
// elimination with the pivot of column j taken among the leaf's rows not taken before
// (largest magnitude; the lowest row of the input on ties).  Rows stay where they are
// while the elimination runs: lane r of every wavefront holds row r, wavefront q its
// columns CW q .. CW q + CW - 1, in registers.  The wavefront that owns column j picks the
// pivot row, leaves the multipliers and then the row's number in LDS, in places of their own
// for every step, and goes on with its next column at once; the wavefronts with later columns
// follow at their own pace, each waiting for a step's row number (a wavefront's LDS
// operations complete in the order they were issued, so the multipliers are there when the
// number is) and reading the pivot row's entries of its own columns from the pivot lane's
// registers.  No step has a barrier, and a wavefront is through with the earlier columns
// about one LDS round trip after their owner.  Every wait ends: the owner of a column waits
// only for earlier columns, and all wavefronts of the one workgroup are on the compute unit.
// The rows are put into the order of their choice at the end.  On return Pl holds L below the
// diagonal and D on it, Qu holds U^T
// (strictly lower, unit diagonal implied), dvec / dinv the pivots and their reciprocals,
// linvL / linvU the inverses of the 16 x 16 diagonal sub-blocks of L and of U^T (for
// leaf_solve_kernel: rows below in Pl are solved against U^T, rows below in Qu against L
// with the leaf's row order as their column gather), perm[j] = pivot0 + (row of the leaf
// taken at step j); flags->odd_leaves is raised by one if that order is an odd permutation.
// Bound by the owner's chain: search 230 clocks (exchanges, a ballot), quotient 70, the next column's
// update 100.  Measured, fp64, inside panel_flow_kernel: 14.8 us a leaf, 25.0 from one leaf to the next (27.4 with the tiles
// left of the leaf stored in front of it and the leaves that they are solved against brought to LDS one after
// the other; n = 2900 1.375 -> 1.282 ms).
// IN_LDS, THROUGH: as for leaf_factor_body; `lds` has LU_LDS_ELEMS elements, of which with IN_LDS the
// first LEAF_TILE hold the leaf, row stride LEAF_PAD.  beside: what the first wavefront is to do when it is through
// with its columns.
constexpr int LU_WAVES = 8;
constexpr int LU_LDS_ELEMS = LEAF_TILE + LEAF * LEAF + LEAF;
template <typename T, int NW, bool IN_LDS = false, bool THROUGH = false, typename Beside = LeafBeside>
__device__ __forceinline__ void leaf_lu_body(
    T* __restrict__ Pl, T* __restrict__ Qu, int64_t ld, int w, T* __restrict__ dvec,
    T* __restrict__ dinv, T* __restrict__ linvL, T* __restrict__ linvU, int* __restrict__ perm,
    long long pivot0, DevFlags* flags, T* __restrict__ lds, const Beside& beside = Beside{}) {
  constexpr int CW = LEAF / NW;          // columns per wavefront
  static_assert(NW == 2 * NSUB, "one diagonal sub-block of L or U^T to invert per wavefront");
  T* const S = lds;                      // the leaf; afterwards, rows in pivot order: L below, D U on and above
  T (* const mult)[LEAF] = reinterpret_cast<T (*)[LEAF]>(S + LEAF_TILE);   // minus the multipliers of every step, by input row
  int* const row_of = reinterpret_cast<int*>(S + LEAF_TILE + LEAF * LEAF); // row taken at a step; -1: not yet
  __builtin_amdgcn_s_setprio(2);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c0 = wave * CW;
  if constexpr (!IN_LDS) {
    // rows of both halves, one row a load: (r, c) of the lower half, (c, r) of the upper;
    // the padding of a narrow leaf is the identity
    T p[CW], q[CW];
#pragma unroll
    for (int k = 0; k < CW; ++k) {
      const int r = NW * k + wave;
      p[k] = (r < w && lane <= r) ? Pl[(int64_t)r * ld + lane] : (r == lane ? T(1) : T(0));
      q[k] = (r < w && lane < r) ? Qu[(int64_t)r * ld + lane] : T(0);
    }
#pragma unroll
    for (int k = 0; k < CW; ++k) {
      const int r = NW * k + wave;
      if (lane <= r) S[r * LEAF_PAD + lane] = p[k];
      if (lane < r) S[lane * LEAF_PAD + r] = q[k];
    }
  }
  if (tid < LEAF) row_of[tid] = -1;
  __syncthreads();
  T a[CW];
#pragma unroll
  for (int k = 0; k < CW; ++k) a[k] = S[lane * LEAF_PAD + c0 + k];
  // rows still to be taken: those of the leaf, and when there are none left (w < 64) those of the padding,
  // whose pivots are their own ones and eliminate nothing
  unsigned long long left = w < LEAF ? (1ull << w) - 1ull : ~0ull;
  const unsigned long long padding = ~left;
  int odd = 0;                           // parity of the row order so far (the last wavefront's)
  auto take = [&](const int p) { left &= ~(1ull << p); };
  auto refill = [&] { left = left != 0ull ? left : padding; };
  auto count = [&](const int p) { odd ^= __popcll(left & ((1ull << p) - 1ull)) & 1; };   // rows to come that stand before p
  // the earlier columns' steps
  auto follow = [&](auto last_tag) {
#pragma unroll 1
    for (int j = 0; j < c0; ++j) {
      lds_volatile<int>* number = (lds_volatile<int>*)&row_of[j];
      lds_volatile<T>* from = (lds_volatile<T>*)&mult[j][lane];
      int p;
      T nl;
      do {
        p = *number;
        nl = *from;
        p = __builtin_amdgcn_readfirstlane(p);
      } while (p < 0);
      T pv[CW];
#pragma unroll
      for (int k = 0; k < CW; ++k) pv[k] = lane_value(a[k], p);
#pragma unroll
      for (int k = 0; k < CW; ++k) a[k] = fma(nl, pv[k], a[k]);
      refill();
      if constexpr (decltype(last_tag)::value) count(p);
      take(p);
    }
  };
  if (wave == NW - 1) follow(std::true_type{});
  else follow(std::false_type{});
  // its own
  __builtin_amdgcn_s_setprio(3);
  int ps[CW];
  const unsigned long long before = left;
  lds_volatile<T>* const mult_to = (lds_volatile<T>*)&mult[c0][lane];
  lds_volatile<int>* const row_to = (lds_volatile<int>*)&row_of[c0];
#pragma unroll
  for (int jj = 0; jj < CW; ++jj) {
    const T cj = a[jj];
    refill();
    const int p = pick_lane(cj, left);
    const T d = lane_value(cj, p);
    const T est = rcp_estimate(d), tail = quotient_tail(d, est);
    take(p);
    const bool below = __builtin_amdgcn_inverse_ballot_w64(left);
    const T np = -(cj * est);
    const T nl = below ? fma(np, tail, np) : T(0);
    mult_to[jj * LEAF] = nl;
    row_to[jj] = p;                                        // (every lane: the same value)
#pragma unroll
    for (int k = jj + 1; k < CW; ++k) a[k] = fma(nl, lane_value(a[k], p), a[k]);
    a[jj] = below ? -nl : cj;
    ps[jj] = p;
  }
  __builtin_amdgcn_s_setprio(2);
  if (wave == 0) beside();
  if (wave == NW - 1) {
    left = before;
#pragma unroll
    for (int jj = 0; jj < CW; ++jj) {
      refill();
      count(ps[jj]);
      take(ps[jj]);
    }
    if (lane == 0 && odd) atomicAdd(&flags->odd_leaves, 1ull);
  }
  __syncthreads();
  {
    // the step at which this row was taken: every lane's number to the lane of its row
    const int to = __builtin_amdgcn_ds_permute(4 * row_of[lane], lane);
#pragma unroll
    for (int k = 0; k < CW; ++k) S[to * LEAF_PAD + c0 + k] = a[k];
  }
  __syncthreads();
  const T myd = S[lane * LEAF_PAD + lane];
  const T myr = fast_rcp(myd);
  T up[CW];
  // L below the diagonal, D on it; U = D U~, transposed
#pragma unroll
  for (int k = 0; k < CW; ++k) {
    a[k] = S[(NW * k + wave) * LEAF_PAD + lane];
    up[k] = S[lane * LEAF_PAD + NW * k + wave] * myr;
  }
#pragma unroll
  for (int k = 0; k < CW; ++k) {
    const int r = NW * k + wave;
    if (r < w && lane <= r) leaf_store<THROUGH>(Pl + (int64_t)r * ld + lane, a[k]);
    if (r < w && lane < r) leaf_store<THROUGH>(Qu + (int64_t)r * ld + lane, up[k]);
  }
  // the inverses of the diagonal sub-blocks, L by the first wavefronts, U~^T by the others
  if (THROUGH) {
  } else if (wave < NSUB) {
    leaf_invert_sub<T>(S, linvL, wave, lane);
  } else {
    const int b = wave - NSUB, c = lane & 15;
    T nl[SUB];
#pragma unroll
    for (int k = 0; k < SUB; ++k) nl[k] = S[(b * SUB + k) * LEAF_PAD + b * SUB + c] * lane_value(myr, b * SUB + k);
#pragma unroll
    for (int k = 0; k < SUB; ++k) nl[k] = c > k ? -nl[k] : T(0);
    invert16<T>(nl, linvU + b * SUB * SUB, lane);
  }
  if (wave == 0) {
    const bool zero = myd == T(0);
    const bool finite = fabs((double)myd) <= 1.7976931348623157e308;
    const bool bad = lane < w && (zero || !finite);
    if (lane < w) {
      leaf_store<THROUGH>(dvec + lane, myd);
      leaf_store<THROUGH>(dinv + lane, myr);
      leaf_store<THROUGH>(perm + lane, (int)pivot0 + row_of[lane]);
    }
    const unsigned long long mask = __ballot(bad);
    if (mask != 0ull) {
      const int first = __ffsll((long long)mask) - 1;
      if (lane == first) {
        unsigned long long idx = (unsigned long long)(pivot0 + first);
        unsigned long long old = atomicMin(&flags->first_bad, idx);
        if (idx <= old) atomicExch(&flags->bad_kind, zero ? 1ull : 2ull);
      }
    }
  }
  __builtin_amdgcn_s_setprio(0);
}

template <typename T, int NW>
__global__ __launch_bounds__(64 * NW) void leaf_lu_kernel(
    T* __restrict__ Pl, T* __restrict__ Qu, int64_t ld, int w, T* __restrict__ dvec,
    T* __restrict__ dinv, T* __restrict__ linvL, T* __restrict__ linvU, int* __restrict__ perm,
    long long pivot0, DevFlags* flags) {
  __shared__ T lds[LU_LDS_ELEMS];
  leaf_lu_body<T, NW>(Pl, Qu, ld, w, dvec, dinv, linvL, linvU, perm, pivot0, flags, lds);
}

// Moves the strict upper triangle of a general matrix into its transposed store, or back,
// by 64 x 64 blocks through LDS (both arrays n x n with leading dimension ld).
// back = 0: dst[i][j] = src[j][i] for i > j;  back = 1: dst[j][i] = src[i][j] for i > j.
// Workgroup b handles the block pair (bi, bj), bi >= bj, of the lower triangle.
template <typename T>
__global__ __launch_bounds__(256) void transpose_strict_kernel(const T* __restrict__ src,
                                                               T* __restrict__ dst, int64_t ld,
                                                               int64_t n, int nb, int back) {
  __shared__ T t[LEAF * LEAF_PAD];
  const int64_t b = blockIdx.x;
  int64_t bi = (int64_t)((sqrt(8.0 * (double)b + 1.0) - 1.0) * 0.5);
  while (bi * (bi + 1) / 2 > b) --bi;
  while ((bi + 1) * (bi + 2) / 2 <= b) ++bi;
  const int64_t bj = b - bi * (bi + 1) / 2;
  if (bi >= nb) return;
  // the block that is read and the block that is written: (row block, column block)
  const int64_t sr = back ? bi : bj, sc = back ? bj : bi;
  const int tid = threadIdx.x;
  for (int e = tid; e < LEAF * LEAF; e += 256) {
    const int r = e >> 6, c = e & 63;
    const int64_t gr = sr * LEAF + r, gc = sc * LEAF + c;
    t[r * LEAF_PAD + c] = (gr < n && gc < n) ? src[gr * ld + gc] : T(0);
  }
  __syncthreads();
  for (int e = tid; e < LEAF * LEAF; e += 256) {
    const int r = e >> 6, c = e & 63;                       // of the block written, (sc, sr)
    const int64_t gr = sc * LEAF + r, gc = sr * LEAF + c;
    const bool strict = back ? gc > gr : gr > gc;
    if (gr < n && gc < n && strict) dst[gr * ld + gc] = t[c * LEAF_PAD + r];
  }
}

// ---------------------------------------------------------------------------
// leaf solve
// ---------------------------------------------------------------------------
// Rows below a factored leaf: X (m x w, in place) <- X L^-T D^-1.
// 256 threads = 4 wavefronts, each owning 16 rows, row r in lane r of every row of 16 lanes;
// row g of lanes has columns 4 g .. 4 g + 3 of each 16-column sub-block (four consecutive
// entries a load).  Sub-block b:  T_b = X_b - sum_{p<b} W_p L[b,p]^T, then W_b = T_b L_bb^-T
// with the inverse of the unit-lower diagonal sub-block prepared by the factor kernel, then
// L_b = W_b D_b^-1 goes back to memory.  The products are formed transposed, L[b,p] W_p^T and
// so on: what a lane holds of X is then both an accumulator and a right operand of the matrix
// instructions (their output row i stands for column solve_col(i) of the sub-block, and the
// left operands, the leaf's rows, are read in that order), so the sub-blocks follow each other
// in registers.  20 KB of LDS in fp64 for the leaf.  Measured, a launch on average, against
// every change of layout in LDS (60 KB in fp64): fp64 n = 1500 7.1 -> 6.0 us, n = 8192 (beside
// the bulk update) 13.2 -> 8.5, fp32 n = 10000 14.7 -> 8.3.  Alone on 32704 rows 12.0 -> 11.7 us in
// fp64 and 9.2 -> 6.9 in fp32, on 131008 35.2 -> 32.6 (4.1 TB/s: bound by memory there) and 23.5 -> 17.8.
// perm (or null): the leaf was factored with pivoting; perm[j] - perm0 is the column of
// the panel that belongs at position j.  A wavefront reads all 64 columns of its rows
// before it writes any of them.
constexpr int SOLVE_ROWS = 64;   // rows per workgroup

// Column of a sub-block that output row i of a 16 x 16 product stands for: accumulator register
// r of row g of lanes holds output row acc_row, and column 4 g + r.
template <typename T> __device__ __forceinline__ int solve_col(int i);
template <> __device__ __forceinline__ int solve_col<double>(int i) { return 4 * (i & 3) + (i >> 2); }
template <> __device__ __forceinline__ int solve_col<float>(int i) { return i; }

// Four consecutive entries (aligned to an entry only: the memory system takes it).
template <typename T>
__device__ __forceinline__ void load4(const T* p, T (&v)[4]) {
  typedef T four __attribute__((ext_vector_type(4), aligned(sizeof(T))));
  const four f = *reinterpret_cast<const four*>(p);
#pragma unroll
  for (int e = 0; e < 4; ++e) v[e] = f[e];
}
template <typename T>
__device__ __forceinline__ void store4(T* p, const T (&v)[4]) {
  typedef T four __attribute__((ext_vector_type(4), aligned(sizeof(T))));
  *reinterpret_cast<four*>(p) = four{v[0], v[1], v[2], v[3]};
}
// A lane's four of every sub-block of a row that starts at p: columns 16 b + 4 g + e < w, the
// others zero.  Whole rows (w = LEAF, the same in all lanes) have a path of their own, in which
// the loads follow each other with nothing in between: with a condition on each of them a solve of
// 131008 rows took 36.4 us in fp64 and 26.0 in fp32, now 32.6 and 17.8.
template <typename T>
__device__ __forceinline__ void load_row(const T* p, const int g, const int w, T (&v)[NSUB][4]) {
  if (w >= LEAF) {
#pragma unroll
    for (int b = 0; b < NSUB; ++b) load4(p + b * SUB + 4 * g, v[b]);
  } else {
#pragma unroll
    for (int b = 0; b < NSUB; ++b)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int col = b * SUB + 4 * g + e;
        v[b][e] = col < w ? p[col] : T(0);
      }
  }
}
template <typename T>
__device__ __forceinline__ void store_row(T* p, const int g, const int w, const T (&v)[NSUB][4]) {
  if (w >= LEAF) {
#pragma unroll
    for (int b = 0; b < NSUB; ++b) store4(p + b * SUB + 4 * g, v[b]);
  } else {
#pragma unroll
    for (int b = 0; b < NSUB; ++b)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int col = b * SUB + 4 * g + e;
        if (col < w) p[col] = v[b][e];
      }
  }
}

// What every wavefront of a solve needs of the leaf, as left operands: minus L[b, p], p < b, and
// the inverses of the diagonal sub-blocks.  The four wavefronts of a workgroup fetch them
// between them, and keep them in LDS in the order in which they are used, 16 bytes a lane: held
// by each wavefront in registers, four times the traffic and 80 registers more, a solve of
// fp64 rows took 7.5 us.
template <typename T>
struct LeafOperands {
  static constexpr int COUNT = NSUB * (NSUB - 1) / 2 + NSUB;      // sub-blocks: minus L, then the inverses
  static constexpr int ELEMS = COUNT * 4 * 64;
  static constexpr int VEC = Mfma<T>::VEC;
  using vec_t = typename Mfma<T>::vec_t;
  T* lds;

  static constexpr int lower(int b, int p) { return b * (b - 1) / 2 + p; }
  // place of entries [VEC h, VEC h + VEC) of this lane's four of sub-block q
  __device__ __forceinline__ vec_t* at(int q, int h, int lane) const {
    return reinterpret_cast<vec_t*>(lds + ((q * (4 / VEC) + h) * 64 + lane) * VEC);
  }
  // this wavefront's share; the caller's barrier publishes it
  __device__ __forceinline__ void stage(const T* __restrict__ Lleaf, int64_t ldl, int w, const T* __restrict__ linv,
                                        const int wave, const int lane) {
    const int g = lane >> 4, row = solve_col<T>(lane & 15);
    T v[3][4];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const int q = 4 * k + wave;
      if (q < COUNT) {
        if (q < COUNT - NSUB) {
          int b = 1;
          while (lower(b + 1, 0) <= q) ++b;
          const int r = b * SUB + row;
          if (r < w) {
            load4(Lleaf + (int64_t)r * ldl + (q - lower(b, 0)) * SUB + 4 * g, v[k]);
          } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) v[k][e] = T(0);
          }
        } else {
          load4(linv + ((q - (COUNT - NSUB)) * SUB + row) * SUB + 4 * g, v[k]);
        }
      }
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const int q = 4 * k + wave;
      const bool minus = q < COUNT - NSUB;
      if (q < COUNT) {
#pragma unroll
        for (int h = 0; h < 4 / VEC; ++h) {
          vec_t o;
#pragma unroll
          for (int e = 0; e < VEC; ++e) o[e] = minus ? -v[k][VEC * h + e] : v[k][VEC * h + e];
          *at(q, h, lane) = o;
        }
      }
    }
  }
  __device__ __forceinline__ void fetch(int q, int lane, T (&v)[4]) const {
#pragma unroll
    for (int h = 0; h < 4 / VEC; ++h) {
      const vec_t o = *at(q, h, lane);
#pragma unroll
      for (int e = 0; e < VEC; ++e) v[VEC * h + e] = o[e];
    }
  }
  // x[b] of 16 rows <- their W_b (undivided)
  __device__ __forceinline__ void solve(typename Mfma<T>::acc_t (&x)[NSUB], const int lane) const {
    using X = Mfma<T>;
    using acc_t = typename X::acc_t;
#pragma unroll
    for (int b = 0; b < NSUB; ++b) {
      T op[4];
#pragma unroll
      for (int p = 0; p < b; ++p) {
        fetch(lower(b, p), lane, op);
#pragma unroll
        for (int s = 0; s < 4; ++s) x[b] = X::mfma(op[s], x[p][s], x[b]);
      }
      fetch(COUNT - NSUB + b, lane, op);
      acc_t wb = acc_t{0, 0, 0, 0};
#pragma unroll
      for (int s = 0; s < 4; ++s) wb = X::mfma(op[s], x[b][s], wb);
      x[b] = wb;
    }
  }
};

template <typename T>
__device__ __forceinline__ void leaf_solve_body(
    T* __restrict__ Xg, int64_t ld, int m, int w, const T* __restrict__ Lleaf, int64_t ldl,
    const T* __restrict__ dinv, const T* __restrict__ linv, const int* __restrict__ perm, int perm0) {
  using acc_t = typename Mfma<T>::acc_t;
  __builtin_amdgcn_s_setprio(2);                // on the chain of dependent launches
  __shared__ __attribute__((aligned(16))) T lds[LeafOperands<T>::ELEMS];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, g = lane >> 4;

  const int64_t row = ((int64_t)blockIdx.x * 4 + wave) * SUB + l16;
  const bool in = row < m;
  T* xrow = Xg + row * ld;
  acc_t x[NSUB];
  {
    T v[NSUB][4];
#pragma unroll
    for (int b = 0; b < NSUB; ++b)
#pragma unroll
      for (int e = 0; e < 4; ++e) v[b][e] = T(0);
    if (perm == nullptr) {
      if (in) load_row((const T*)xrow, g, w, v);
    } else {
      // column `col` of the result is the column that was taken at that step
#pragma unroll
      for (int b = 0; b < NSUB; ++b)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int col = b * SUB + 4 * g + e;
          if (in && col < w) v[b][e] = xrow[perm[col] - perm0];
        }
    }
#pragma unroll
    for (int b = 0; b < NSUB; ++b)
#pragma unroll
      for (int e = 0; e < 4; ++e) x[b][e] = v[b][e];
  }
  LeafOperands<T> ops{lds};
  ops.stage(Lleaf, ldl, w, linv, wave, lane);
  T rinv[NSUB][4];
  load_row(dinv, g, w, rinv);
  __syncthreads();
  // with a permutation a store below may hit an entry that another lane of this wavefront
  // loads above: every load has returned before the first store is issued
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  ops.solve(x, lane);
  if (in) {
    T v[NSUB][4];
#pragma unroll
    for (int b = 0; b < NSUB; ++b)
#pragma unroll
      for (int e = 0; e < 4; ++e) v[b][e] = x[b][e] * rinv[b][e];
    store_row(xrow, g, w, v);
  }
}

template <typename T>
__global__ __launch_bounds__(256) void leaf_solve_kernel(
    T* __restrict__ Xg, int64_t ld, int m, int w, const T* __restrict__ Lleaf, int64_t ldl,
    const T* __restrict__ dinv, const T* __restrict__ linv, const int* __restrict__ perm, int perm0) {
  leaf_solve_body<T>(Xg, ld, m, w, Lleaf, ldl, dinv, linv, perm, perm0);
}

// The rows below a leaf of a general matrix, both halves in one launch with two rows of
// workgroups: blockIdx.y = 0 solves the rows of the lower half (Xg) against U^T (the leaf's
// place in the second array, qoff elements on) with linvU; blockIdx.y = 1 the rows of the
// transposed upper half (Xg + qoff) against L (Lleaf) with linvL, their columns gathered
// in the leaf's row order (perm, perm0 as in leaf_solve_kernel).
template <typename T>
__global__ __launch_bounds__(256) void leaf_solve_general_kernel(
    T* Xg, int64_t ld, int m, int w, const T* Lleaf, const T* __restrict__ dinv,
    const T* __restrict__ linvL, const T* __restrict__ linvU, const int* __restrict__ perm, int perm0, int64_t qoff) {
  const bool upper = blockIdx.y != 0;
  leaf_solve_body<T>(upper ? Xg + qoff : Xg, ld, m, w, upper ? Lleaf : Lleaf + qoff, ld, dinv,
                     upper ? linvL : linvU, upper ? perm : (const int*)nullptr, perm0);
}

}  // namespace mdet
