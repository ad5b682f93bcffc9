// Symmetric pivoting over a whole diagonal block (MDET_FLAG_PIVOT_BLOCK).
//
// Sec. 2.2 of the paper: the symmetric form handles permutations, pivoting is done inside
// each block and not between blocks; the software appendix returns `perm` with
// P^T M P = L D L^T.  Here the candidates of every elimination step are ALL entries left
// on the diagonal of the current Schur complement inside the block column's w x w diagonal
// block (the 64-column leaf of MDET_FLAG_PIVOT is the special case w = 64); the pivot is
// the one of largest magnitude, the one that came first in the input on ties, a NaN counts
// as the largest.  D stays diagonal (1 x 1 pivots only).
//
// A pivot anywhere in the block needs that candidate's column up to date with every pivot
// taken before it.  The scheme is the blocked one with a running diagonal: the diagonal
// block is kept as a full symmetric matrix S in the workspace, brought up to date with 64
// pivots at a time (one product S -= L_p D L_p^T on the matrix cores); inside such a group
// of 64 a step works on the block's rows,
//     v_i   = S[p][i] - sum_{k < j, this group} L[i][k] (d_k L[p][k])      (column of pivot p)
//     l_ij  = v_i / d_j,      d_j = running diagonal of p,
//     diag_i <- diag_i - l_ij v_i,
// all steps in one launch where one workgroup holds the block's rows (pb_group_kernel), one
// small launch a step otherwise, which leaves the partial maxima from which the next one
// picks its pivot (pb_step_kernel).  Nothing is swapped while the block is eliminated: rows keep their input positions, columns are in
// pivot order (`Lfull`), and the rows below the diagonal block get their 64 new columns by
// a gather of the pivots' columns, a product with everything solved before (matrix cores),
// and the leaf solve of the unpivoted path.  At the end the factor is put in place in
// pivot order.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kernels_leaf.h"
#include "kernels_update.h"

namespace mdet {

constexpr int PB_THREADS = 256;

// A candidate: magnitude as its bit pattern (IEEE magnitudes order like their patterns; NaN
// mapped to the pattern of infinity plus one so that it wins), and the row; no candidate: key 0.
struct PbCand {
  unsigned long long key;
  long long row;
};

__device__ __forceinline__ unsigned long long pb_key(double v) {
  if (!(v == v)) return 0x7ff0000000000001ull;
  return (unsigned long long)__double_as_longlong(fabs(v)) + 1ull;     // +1: a zero is still a candidate
}
__device__ __forceinline__ unsigned long long pb_key(float v) {
  if (!(v == v)) return 0x7f800001ull;
  return (unsigned long long)(unsigned)__float_as_int(fabsf(v)) + 1ull;
}
// larger magnitude wins, the smaller row on ties
__device__ __forceinline__ bool pb_better(const PbCand& a, const PbCand& b) {
  return a.key > b.key || (a.key == b.key && a.key != 0ull && a.row < b.row);
}

// Best candidate of the workgroup, in every thread.  s: PB_THREADS entries of LDS.
__device__ __forceinline__ PbCand pb_block_best(PbCand mine, PbCand* s) {
  s[threadIdx.x] = mine;
  __syncthreads();
  for (int h = PB_THREADS / 2; h > 0; h >>= 1) {
    if ((int)threadIdx.x < h && pb_better(s[threadIdx.x + h], s[threadIdx.x])) s[threadIdx.x] = s[threadIdx.x + h];
    __syncthreads();
  }
  const PbCand r = s[0];
  __syncthreads();
  return r;
}

// S <- the w x w diagonal block as a full symmetric matrix (only its lower triangle is read
// from P): 32 x 32 tiles on and below the diagonal, each written straight and transposed
// through LDS so that both the reads and the writes run along rows.  Grid: (tiles per side)^2.
template <typename T>
__global__ __launch_bounds__(256) void pb_symmetrize_kernel(const T* __restrict__ P, int64_t ld, int w,
                                                            T* __restrict__ S, int64_t lds) {
  __shared__ T t[32][33];
  const int nt = (w + 31) / 32;
  const int bi = blockIdx.x / nt, bj = blockIdx.x % nt;
  if (bj > bi) return;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;         // 32 x 8
  for (int r = ty; r < 32; r += 8) {
    const int gr = bi * 32 + r, gc = bj * 32 + tx;
    T v = T(0);
    if (gr < w && gc < w) v = gc <= gr ? P[(int64_t)gr * ld + gc] : P[(int64_t)gc * ld + gr];
    t[r][tx] = v;
    if (gr < w && gc < w) S[(int64_t)gr * lds + gc] = v;
  }
  __syncthreads();
  if (bi != bj)
    for (int r = ty; r < 32; r += 8) {
      const int gr = bj * 32 + r, gc = bi * 32 + tx;            // the mirrored tile
      if (gr < w && gc < w) S[(int64_t)gr * lds + gc] = t[tx][r];
    }
}

// The running diagonal, all rows candidates, columns w .. ldl of Lfull zero, and the first
// step's partial maxima.
template <typename T>
__global__ __launch_bounds__(PB_THREADS) void pb_init_kernel(const T* __restrict__ P, int64_t ld, int w,
                                                             T* __restrict__ Lfull, int64_t ldl,
                                                             T* __restrict__ dg, int* __restrict__ active,
                                                             PbCand* __restrict__ part) {
  __shared__ PbCand red[PB_THREADS];
  const int i = blockIdx.x * PB_THREADS + threadIdx.x;
  PbCand mine{0ull, 0};
  if (i < w) {
    const T d = P[(int64_t)i * ld + i];
    dg[i] = d;
    active[i] = 1;
    mine = PbCand{pb_key(d), i};
    for (int64_t c = w; c < ldl; ++c) Lfull[(int64_t)i * ldl + c] = T(0);
  }
  const PbCand best = pb_block_best(mine, red);
  if (threadIdx.x == 0) part[blockIdx.x] = best;
}

// One elimination step: step jj of the group of 64 that starts at column c0 (pivot order).
template <typename T>
__global__ __launch_bounds__(PB_THREADS) void pb_step_kernel(
    const T* __restrict__ S, int64_t lds, T* __restrict__ Lfull, int64_t ldl, T* __restrict__ dg,
    int* __restrict__ active, const PbCand* __restrict__ part_in, PbCand* __restrict__ part_out, int nparts,
    int* __restrict__ piv, T* __restrict__ dvec, T* __restrict__ dinv, int* __restrict__ perm, int w, int c0,
    int jj, long long pivot0, DevFlags* flags) {
  __shared__ PbCand red[PB_THREADS];
  __shared__ T wrow[LEAF];
  // the pivot: best of the partial maxima the step before left (every workgroup finds it alone)
  PbCand mine{0ull, 0};
  for (int q = threadIdx.x; q < nparts; q += PB_THREADS)
    if (pb_better(part_in[q], mine)) mine = part_in[q];
  const PbCand top = pb_block_best(mine, red);
  const int p = (int)top.row;
  const T d = dg[p];
  // the pivot row's entries of this group, times their pivots: w_k = d_k L[p][k]
  if ((int)threadIdx.x < jj) wrow[threadIdx.x] = Lfull[(int64_t)p * ldl + c0 + threadIdx.x] * dvec[c0 + threadIdx.x];
  __syncthreads();
  const int i = blockIdx.x * PB_THREADS + threadIdx.x;
  PbCand next{0ull, 0};
  if (i < w) {
    T l = T(0);
    if (active[i] != 0 && i != p) {
      T v = S[(int64_t)p * lds + i];
      const T* Li = Lfull + (int64_t)i * ldl + c0;
      for (int k = 0; k < jj; ++k) v = fma(-Li[k], wrow[k], v);
      l = v / d;
      const T nd = fma(-l, v, dg[i]);
      dg[i] = nd;
      next = PbCand{pb_key(nd), i};
    }
    Lfull[(int64_t)i * ldl + c0 + jj] = l;
    if (i == p) {
      active[i] = 0;
      piv[c0 + jj] = p;
      dvec[c0 + jj] = d;
      dinv[c0 + jj] = T(1) / d;
      perm[c0 + jj] = (int)pivot0 + p;
      const bool zero = d == T(0);
      const bool finite = fabs((double)d) <= 1.7976931348623157e308;
      if (zero || !finite) {
        const unsigned long long idx = (unsigned long long)(pivot0 + c0 + jj);
        const unsigned long long old = atomicMin(&flags->first_bad, idx);
        if (idx <= old) atomicExch(&flags->bad_kind, zero ? 1ull : 2ull);
      }
    }
  }
  const PbCand best = pb_block_best(next, red);
  if (threadIdx.x == 0) part_out[blockIdx.x] = best;
}

// All steps of a group of up to 64 pivots in one launch of one workgroup, thread i holding
// row i (w <= NT): its running diagonal and its multipliers of this group stay in registers.
// The rows of S that the group is likely to take, those of the largest diagonal entries as it begins,
// are brought into LDS first, and their multipliers kept there.  Per step: every wavefront's best candidate
// to LDS; one barrier; the overall best found by every thread alone; its row of S and multipliers from
// LDS, or from memory and the row's thread where another row than expected is taken; then v, l and the new diagonal as in pb_step_kernel, with
// the products of a block of multipliers taking the pivot's entries from the lanes of the row (one
// instruction each).  At the end the group's leaf, in pivot order, with the inverses of its diagonal
// sub-blocks (as pb_leaf_kernel).  Same rule, same order of the terms as a sequence of
// pb_step_kernel launches, where a launch and its memory round trips made a step 5.7 us.
// Bound by a step's chain, w = 256, fp64: search 150 clocks, offer and barrier 140, best of the offers 190, row and
// multipliers from LDS 150, products 370, quotient and the rest 200: 0.65 us.  A launch of 64 steps 43.5 us; 71 with the row
// of S from memory (1100 clocks), a second barrier for the pivot's multipliers and a dozen jumps a step
// (n = 3000, ms, b = 256 and 512: fp64 4.82 -> 3.40, 5.85 -> 4.32, fp32 4.04 -> 2.82, 4.36 -> 3.03; where half of the
// rows taken are not held, b = 256, 4.82 -> 3.81).
// The multipliers of 512 rows are what a compute unit's registers hold (128 of 256 per
// thread in fp64): larger blocks take a launch per step.
constexpr int PB_GROUP_ROWS = 512;

// Magnitudes as integers that order alike (a NaN above all others).
__device__ __forceinline__ unsigned long long pb_magnitude(double v) {
  return (unsigned long long)__double_as_longlong(v) & 0x7fffffffffffffffull;
}
__device__ __forceinline__ unsigned long long pb_magnitude(float v) { return __float_as_uint(v) & 0x7fffffffu; }

// A power of two that brings d away from the ends of its range if it is there.
__device__ __forceinline__ double pb_lift(double d) {
  const unsigned e = ((unsigned)__double2hiint(d) >> 20) & 0x7ffu;
  return __hiloint2double(e == 0u ? 0x46700000 : (e > 0x7fbu ? 0x39700000 : 0x3ff00000), 0);      // 2^104, 2^-104, 1
}
__device__ __forceinline__ float pb_lift(float d) {
  const unsigned e = (__float_as_uint(d) >> 23) & 0xffu;
  return __uint_as_float(e == 0u ? 0x56800000u : (e > 0xfbu ? 0x28800000u : 0x3f800000u));        // 2^46, 2^-46, 1
}

// What a wavefront offers as the pivot: its value; its row, and its place in LDS (or -1) from bit 16 on;
// the upper word of its magnitude plus one (no candidate: 0).
struct alignas(16) PbOffer {
  unsigned lo, hi;
  int row;
  unsigned rank;
};
__device__ __forceinline__ PbOffer pb_offer(double v, int row, bool any) {
  const unsigned hi = (unsigned)__double2hiint(v);
  return {(unsigned)__double2loint(v), hi, row, any ? (hi & 0x7fffffffu) + 1u : 0u};
}
__device__ __forceinline__ PbOffer pb_offer(float v, int row, bool any) {
  return {0u, __float_as_uint(v), row, any ? (__float_as_uint(v) & 0x7fffffffu) + 1u : 0u};
}
__device__ __forceinline__ void pb_value(const PbOffer& o, int q, double& d) {
  d = __hiloint2double(__builtin_amdgcn_readlane((int)o.hi, q), __builtin_amdgcn_readlane((int)o.lo, q));
}
__device__ __forceinline__ void pb_value(const PbOffer& o, int q, float& d) {
  d = __int_as_float(__builtin_amdgcn_readlane((int)o.hi, q));
}
// The best of NW offers, offer l % NW in lane l: larger magnitude wins, the first on ties (which has
// the smaller row).
template <typename T, int NW>
__device__ __forceinline__ int pb_best(const PbOffer& o) {
  unsigned m = o.rank;
  m = max(m, (unsigned)__builtin_amdgcn_update_dpp(0, (int)m, 0xB1, 0xF, 0xF, false));     // lanes 1 0 3 2 of each four
  m = max(m, (unsigned)__builtin_amdgcn_update_dpp(0, (int)m, 0x4E, 0xF, 0xF, false));     // lanes 2 3 0 1
  if (NW == 8) m = max(m, (unsigned)__builtin_amdgcn_update_dpp(0, (int)m, 0x141, 0xF, 0xF, false));   // mirror inside each eight
  unsigned hit = (unsigned)__builtin_amdgcn_ballot_w64(o.rank == m) & ((1u << NW) - 1u);
  if (sizeof(T) == 8 && __builtin_expect((hit & (hit - 1u)) != 0u, 0)) {
    const bool level = __builtin_amdgcn_inverse_ballot_w64((unsigned long long)hit);
    const unsigned top = wave_max_u32(level ? o.lo : 0u);
    hit &= (unsigned)__builtin_amdgcn_ballot_w64(o.lo == top);
  }
  return __builtin_ctz(hit);
}

// Rows of S that LDS holds, with their multipliers: all 64 that a group takes where they fit (fp32); in fp64 as many as
// there is room for, 62 of blocks up to 256 and 34 of wider ones.
template <typename T, int NT>
struct PbHeld {
  static constexpr int ROOM = 156 * 1024 / (int)sizeof(T);
  static constexpr int HELD = 64 * NT + LEAF * 65 <= ROOM ? 64 : (ROOM - LEAF) / (NT + LEAF) / 2 * 2;
  static constexpr int STRIDE = HELD + 1;        // (column HELD: of rows that are not held)
  T rows[HELD * NT];                             // at the end the group's leaf
  T mult[LEAF * STRIDE];                         // multipliers, by step
  T other[SUB];                                  // the last ones of a row that is not held
  PbOffer offer[2][NT / 64];                     // every wavefront's best candidate; two steps in turn
  int place[HELD];
};

// A thread's row in a group of steps.
template <typename T, int NT>
struct PbRow {
  using H = PbHeld<T, NT>;
  static constexpr int NW = NT / 64;
  H& s;
  const T* S;
  const int64_t lds;
  const T* L;                                    // this group's columns of Lfull
  const int64_t ldl;
  const int w, lw;
  const int i, lane, l16, wave;
  int place;                                     // in s, or -1
  T* own;                                        // its column of s.mult
  T diag;
  unsigned long long left;                       // the wavefront's rows that are still to be taken
  int mypos = -1;                                // step at which this row was taken
  // multipliers of the finished blocks of 16 steps and of the current one (0: not taken yet);
  // pivots and rows likewise, step k of a block in lane k of each row of lanes
  T h[3][SUB], cur[SUB], dh[3], dcur;
  int pcur;

  // 16 steps, the M-th block of them (known at compile time, like the step in it: a jump on either costs
  // a step some 25 clocks, and there were a dozen)
  template <int M>
  __device__ __forceinline__ void block() {
#pragma unroll
    for (int k = 0; k < SUB; ++k) cur[k] = T(0);
    dcur = T(0);
    pcur = 0;
    int mine = l16;
    asm volatile("" : "+v"(mine));               // compared here, not kept as 16 masks in scalar registers
#pragma unroll
    for (int j = 0; j < SUB; ++j) {
      constexpr int J0 = SUB * M;
      const int par = j & 1;
      if (J0 + j >= lw) break;
      const int best = pick_lane(diag, left);
      // (what the step before last left in these places has been read: its readers are through a barrier)
      if (lane == best) s.offer[par][wave] = pb_offer(diag, i | (place << 16), left != 0ull);
      __syncthreads();
      const PbOffer o = s.offer[par][lane & (NW - 1)];
      const int win = pb_best<T, NW>(o);
      T d;
      pb_value(o, win, d);
      const int taken = __builtin_amdgcn_readlane(o.row, win);
      const int p = taken & 0xffff, at = taken >> 16;          // at: -1 if it is not held
      const int from = at < 0 ? 0 : at;
      T wk[M + 1], v = s.rows[from * NT + i];
#pragma unroll
      for (int b = 0; b <= M; ++b) wk[b] = s.mult[(SUB * b + l16) * H::STRIDE + from];
      if (__builtin_expect(at < 0, 0)) {
        v = i < w ? S[(int64_t)p * lds + i] : T(0);
#pragma unroll
        for (int b = 0; b < M; ++b) wk[b] = L[(int64_t)p * ldl + SUB * b + l16];
        if (i == p) {
#pragma unroll
          for (int k = 0; k < SUB; ++k) s.other[k] = cur[k];
        }
        __syncthreads();
        wk[M] = s.other[l16];
      }
      // meanwhile the reciprocal, of a pivot that has been brought away from the ends of the range if
      // it was there (the reciprocal of one in the last binades is infinite or subnormal)
      const T lift = pb_lift(d);
      const T dl = d * lift;
      const T rd = fast_rcp(dl);
      mypos = i == p ? J0 + j : mypos;
      left &= ~(p >> 6 == wave ? 1ull << (p & 63) : 0ull);
#pragma unroll
      for (int b = 0; b < M; ++b) apply_first(v, h[b], wk[b] * dh[b], SUB);
      apply_first(v, cur, wk[M] * dcur, j);
      dcur = mine == j ? d : dcur;
      pcur = mine == j ? p : pcur;
      // v / d: the product with the reciprocal, and one correction
      const T vl = v * lift, q = vl * rd;
      const T l = __builtin_amdgcn_inverse_ballot_w64(left) ? fma(fma(-dl, q, vl), rd, q) : T(0);
      diag = fma(-l, v, diag);
      cur[j] = l;
      own[(J0 + j) * H::STRIDE] = l;
    }
  }
};

template <typename T, int NT>
__global__ __launch_bounds__(NT) void pb_group_kernel(const T* __restrict__ S, int64_t lds, T* __restrict__ Lfull,
                                                      int64_t ldl, T* __restrict__ dg, int* __restrict__ active,
                                                      int* __restrict__ piv, T* __restrict__ dvec,
                                                      T* __restrict__ dinv, int* __restrict__ perm, int w, int c0,
                                                      int lw, long long pivot0, DevFlags* flags,
                                                      T* __restrict__ leaf, T* __restrict__ linv) {
  using H = PbHeld<T, NT>;
  constexpr int NW = NT / 64, HELD = H::HELD;
  using vec_t = typename Mfma<T>::vec_t;
  constexpr int VEC = Mfma<T>::VEC;
  __shared__ __attribute__((aligned(16))) H s;
  static_assert(HELD * NT >= LEAF_TILE && HELD * sizeof(T) >= 4, "the leaf's place, and the keys'");
  const int i = threadIdx.x, lane = i & 63;
  const int wave = __builtin_amdgcn_readfirstlane(i >> 6);
  PbRow<T, NT> r{s, S, lds, Lfull + c0, ldl, w, lw, i, lane, i & 15, wave};
  r.diag = i < w ? dg[i] : T(0);
  const bool live = i < w && active[i] != 0;
  r.left = __builtin_amdgcn_ballot_w64(live);
  {
    // places in the order of the magnitudes (their first 22 bits: a guess is all this is)
    typedef unsigned u4 __attribute__((ext_vector_type(4)));
    unsigned* const keys = reinterpret_cast<unsigned*>(s.rows);
    const unsigned top = sizeof(T) == 8 ? (unsigned)((unsigned long long)pb_magnitude(r.diag) >> 32) : (unsigned)pb_magnitude(r.diag);
    const unsigned key = live ? 0x80000000u | (top >> 9 << 9) | (unsigned)(511 - i) : 0u;
    keys[i] = key;
    if (i < HELD) s.place[i] = 0;
    for (int e = i; e < LEAF * H::STRIDE; e += NT) s.mult[e] = T(0);
    __syncthreads();
    int place = 0;
#pragma unroll 4
    for (int q = 0; q < NT; q += 4) {
      const u4 k = *reinterpret_cast<const u4*>(&keys[q]);
      place += (k[0] > key) + (k[1] > key) + (k[2] > key) + (k[3] > key);
    }
    r.place = live && place < HELD ? place : -1;
    r.own = s.mult + (r.place < 0 ? HELD : place);
    if (r.place >= 0) s.place[place] = i;
    __syncthreads();
    // the rows, whole, in pieces of a wavefront's 1 KB (lds is a multiple of 64: a piece of a lane's is in the row or
    // behind its end, where it is anything)
    constexpr int PIECES = NT / (64 * VEC);
    const unsigned at = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)(upd_lds_ptr)s.rows);
    for (int h = wave; h < HELD; h += NW) {
      const char* row = reinterpret_cast<const char*>(S + (int64_t)__builtin_amdgcn_readfirstlane(s.place[h]) * lds);
#pragma unroll
      for (int c = 0; c < PIECES; ++c) {
        const int col = (c * 64 + lane) * VEC;
        load_to_lds<16, 0>(row, (unsigned)((col < lds ? col : 0) * (int)sizeof(T)), at + (unsigned)((h * NT + c * 64 * VEC) * (int)sizeof(T)));
      }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
  }
#pragma unroll
  for (int b = 0; b < 3; ++b) {
    r.dh[b] = T(0);
#pragma unroll
    for (int k = 0; k < SUB; ++k) r.h[b][k] = T(0);
  }
  // what 16 steps have left, to memory
  auto out = [&](const int m) {
    if (i < w) {
      T* to = Lfull + (int64_t)i * ldl + c0 + SUB * m;
#pragma unroll
      for (int k = 0; k < SUB; k += VEC) {
        vec_t v;
#pragma unroll
        for (int e = 0; e < VEC; ++e) v[e] = r.cur[k + e];
        *reinterpret_cast<vec_t*>(to + k) = v;
      }
    }
    if (wave == 0) {
      const int jj = SUB * m + r.l16;
      const T d = r.dcur;
      const bool mine_out = lane < SUB && jj < lw;
      const bool zero = d == T(0);
      const bool finite = fabs((double)d) <= 1.7976931348623157e308;
      if (mine_out) {
        piv[c0 + jj] = r.pcur;
        dvec[c0 + jj] = d;
        dinv[c0 + jj] = T(1) / d;
        perm[c0 + jj] = (int)pivot0 + r.pcur;
      }
      const unsigned long long bad = __builtin_amdgcn_ballot_w64(mine_out && (zero || !finite));
      if (bad != 0ull && lane == __builtin_ctzll(bad)) {
        const unsigned long long idx = (unsigned long long)(pivot0 + c0 + jj);
        const unsigned long long old = atomicMin(&flags->first_bad, idx);
        if (idx <= old) atomicExch(&flags->bad_kind, zero ? 1ull : 2ull);
      }
    }
    if (m < 3) {
      r.dh[m] = r.dcur;
#pragma unroll
      for (int k = 0; k < SUB; ++k) r.h[m][k] = r.cur[k];
    }
  };
  r.template block<0>();
  out(0);
  if (lw > SUB) {
    r.template block<1>();
    out(1);
  }
  if (lw > 2 * SUB) {
    r.template block<2>();
    out(2);
  }
  if (lw > 3 * SUB) {
    r.template block<3>();
    out(3);
  }
  if (i < w) {
    dg[i] = r.diag;
    active[i] = (int)(r.left >> lane & 1ull);
  }
  // the rows taken are rows of the leaf; multipliers behind a row's own step are zero
  T* const tile = s.rows;
  __syncthreads();
  for (int e = i; e < LEAF_TILE; e += NT) tile[e] = T(0);
  __syncthreads();
  if (r.mypos >= 0) {
#pragma unroll
    for (int b = 0; b < 3; ++b)
#pragma unroll
      for (int k = 0; k < SUB; ++k) tile[r.mypos * LEAF_PAD + SUB * b + k] = r.h[b][k];
    if (lw > 3 * SUB) {
#pragma unroll
      for (int k = 0; k < SUB; ++k) tile[r.mypos * LEAF_PAD + 3 * SUB + k] = r.cur[k];
    }
  }
  __syncthreads();
  for (int e = i; e < LEAF * LEAF; e += NT) {
    const int row = e >> 6, col = e & 63;
    leaf[e] = col < row ? tile[row * LEAF_PAD + col] : T(0);
  }
  if (wave < NSUB) leaf_invert_sub<T>(tile, linv, wave, lane);
}

// The group's own lw x lw leaf in pivot order (strictly lower part; 64 x 64, leading
// dimension 64) and the inverses of its 16 x 16 diagonal sub-blocks, as the leaf solve
// wants them.  One workgroup of 256 threads.
template <typename T>
__global__ __launch_bounds__(256) void pb_leaf_kernel(const T* __restrict__ Lfull, int64_t ldl,
                                                      const int* __restrict__ piv, int c0, int lw,
                                                      T* __restrict__ leaf, T* __restrict__ linv) {
  __shared__ T tile[LEAF * LEAF_PAD];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  for (int e = tid; e < LEAF * LEAF; e += 256) {
    const int r = e >> 6, c = e & 63;
    const T v = (r < lw && c < r) ? Lfull[(int64_t)piv[c0 + r] * ldl + c0 + c] : T(0);
    tile[r * LEAF_PAD + c] = v;
    leaf[r * LEAF + c] = v;
  }
  __syncthreads();
  leaf_invert_sub<T>(tile, linv, wave, lane);
}

// Rows below the diagonal block: their columns of the group's pivots, side by side in pivot
// order, into Y[:, c0 .. c0 + 64) (columns past lw zero); and the pivots' own rows of
// everything solved before, Bg[t][0 .. c0) = Lfull[piv[c0 + t]][0 .. c0).
template <typename T>
__global__ __launch_bounds__(256) void pb_gather_kernel(const T* __restrict__ X, int64_t ldx, int64_t rows,
                                                        T* __restrict__ Y, int64_t ldy,
                                                        const T* __restrict__ Lfull, int64_t ldl,
                                                        T* __restrict__ Bg, int64_t ldb,
                                                        const int* __restrict__ piv, int c0, int lw) {
  const int t = threadIdx.x & 63, sub = threadIdx.x >> 6;
  const int src = t < lw ? piv[c0 + t] : 0;
  for (int64_t r = (int64_t)blockIdx.x * 4 + sub; r < rows; r += (int64_t)gridDim.x * 4)
    Y[r * ldy + c0 + t] = t < lw ? X[r * ldx + src] : T(0);
  // the first workgroups also copy the pivots' rows (64 rows of c0 entries)
  for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < (int64_t)LEAF * c0; e += (int64_t)gridDim.x * 256) {
    const int row = (int)(e / c0), k = (int)(e % c0);
    Bg[(int64_t)row * ldb + k] = row < lw ? Lfull[(int64_t)piv[c0 + row] * ldl + k] : T(0);
  }
}

// The factor into its place, in pivot order: unit-lower L of the diagonal block (row r =
// the multipliers of the row taken at step r), D on the diagonal, the rows below from Y.
template <typename T>
__global__ __launch_bounds__(256) void pb_store_kernel(T* __restrict__ P, int64_t ld, int64_t m, int w,
                                                       const T* __restrict__ Lfull, int64_t ldl,
                                                       const int* __restrict__ piv, const T* __restrict__ dvec,
                                                       const T* __restrict__ Y, int64_t ldy) {
  for (int64_t r = blockIdx.x; r < m; r += gridDim.x) {
    if (r < w) {
      const int src = piv[r];
      for (int c = threadIdx.x; c <= r; c += 256)
        P[r * ld + c] = c == r ? dvec[r] : Lfull[(int64_t)src * ldl + c];
    } else {
      for (int c = threadIdx.x; c < w; c += 256) P[r * ld + c] = Y[(r - w) * ldy + c];
    }
  }
}

}  // namespace mdet
