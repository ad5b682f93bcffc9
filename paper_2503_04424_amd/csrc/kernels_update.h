// Trailing Schur-complement update on the matrix cores.
//
// Sec. 2.2 of the paper forms S <- S - C B for every block of the trailing matrix
// (App. E.1 counts it as "full" and "Gramian" matrix multiplications); in the
// LDL^T case the product carries the diagonal scaling:
//
//      C[M x N]  -=  A[M x K] * diag(d[0..K)) * B[N x K]^T
//
// with A and B rows of the already-factored block column (unit-lower factor L)
// and d its pivots.  All three matrices are row-major, so both operands are read
// along K with unit stride.
//
// Tiling (gfx950): 256 threads = 4 wavefronts in a 2 x 2 arrangement, each
// wavefront owns a 64 x 64 piece of a 128 x 128 block of C as 4 x 4 MFMA tiles of
// 16 x 16 (v_mfma_f64_16x16x4_f64 / v_mfma_f32_16x16x4_f32).  K is walked in
// slabs of 128 bytes per row (16 doubles / 32 floats) that go from global memory
// straight into LDS, double buffered, the next slab's loads in flight while the
// current one is multiplied.  The scaling by -d is applied to the A fragments as
// they are read from LDS; the accumulators are seeded with C.
// Bound by the matrix cores.  The wavefronts of a workgroup meet once a slab, in front of its last strip
// of products, behind which nothing of the slab is read any more: the next slab's first fragments and
// the loads of the one after it go out beside those products.  Measured, M = N = 16384, K = 2048, random
// entries, a launch alone: fp64 73.5 TFLOP/s with scaling, 74.5 without (66.6 and 70.0 with the loads in one piece at the
// start of a slab and the meeting at its end), fp32 143.3 and 146.3 (132.8, 137.0); of the 78.6 / 157.3 at
// the matrix cores' peak 4 % go into loading and storing C.
//
// Also here, because it ends with the same hand-over of the next leaf: leaf_update_kernel
// (K = 64, one shot from LDS).
//
// The *_general_kernel names run the same bodies for a general matrix (Sec. 2.2, Eq. 1:
// M = P L U) kept as two lower-triangular arrays, one row of workgroups per array.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "kernels_leaf.h"
#include "mfma.h"

namespace mdet {

constexpr int UPD_THREADS = 256;

// Block scheduling.  The C blocks of a launch are grouped into 8 x 8 "super-tiles"
// (64 blocks that share 8 row strips of A and 8 row strips of B) and numbered
// super-tile by super-tile; of a lower-triangular launch only the blocks on or
// below the diagonal get a number (36 of a super-tile on the diagonal).
// Workgroups are dispatched round-robin over the 8 XCDs by linear id, each XCD
// with its own L2; the map below hands every XCD a contiguous range of block
// numbers, so the 64 or so blocks an XCD runs at one time re-use each operand
// strip eight times out of its L2 instead of fetching it once per block.  Numbers
// that fall outside a ragged edge exit at once.  A launch at most four blocks wide
// (the updates inside a block column) has no use for super-tiles: its blocks are
// numbered row by row.
//
// A launch may cover only part of the numbers: workgroup id takes number
// xcd * per + k0 + (id >> 3) with xcd = id & 7, so that a sequence of launches with
// growing k0 walks every XCD's range in order (used to keep part of the device
// free for the kernels of another stream).
constexpr int UPD_SUPER = 8;
constexpr int UPD_SUPER_LOG2 = 3;

struct UpdGrid {
  int64_t per;       // block numbers per XCD; a full launch has 8 * per workgroups
  int nsn;           // super-tile columns (super-tile mode)
  int swl;           // 3: 8 x 8 super-tiles; 0..2: rows of 1 << swl blocks, no super-tiles
};
static inline UpdGrid update_grid(int64_t M, int64_t N, bool lower, int tile) {
  int64_t nbm = (M + tile - 1) / tile, nbn = (N + tile - 1) / tile;
  UpdGrid g;
  int64_t count;
  if (nbn <= 4) {
    g.swl = nbn <= 1 ? 0 : (nbn <= 2 ? 1 : 2);
    g.nsn = 1;
    count = nbm << g.swl;
  } else {
    g.swl = UPD_SUPER_LOG2;
    const int64_t nsm = (nbm + UPD_SUPER - 1) / UPD_SUPER;
    g.nsn = (int)((nbn + UPD_SUPER - 1) / UPD_SUPER);
    if (!lower) count = nsm * g.nsn * 64;
    else {
      const int64_t t = nsm < g.nsn ? nsm : g.nsn;      // super-tile rows that reach the diagonal
      count = 32 * t * t + 4 * t + (nsm - t) * g.nsn * 64;
    }
  }
  g.per = (count + 7) / 8;
  return g;
}

// (bm, bn) of block number t, or false if there is no such block.  Number 0 is
// block (0, 0).
__host__ __device__ __forceinline__ bool update_block_of_number(const bool lower, const int64_t t, int nbm,
                                                       int nbn, int nsn, int swl, int& bm, int& bn) {
  if (swl < UPD_SUPER_LOG2) {
    bm = (int)(t >> swl);
    bn = (int)(t & ((1 << swl) - 1));
    return bm < nbm && bn < nbn && (!lower || bn <= bm);
  }
  if (!lower) {
    const int64_t st = t >> 6;
    const int loc = (int)(t & 63);
    bm = (int)(st / nsn) * UPD_SUPER + (loc >> 3);
    bn = (int)(st % nsn) * UPD_SUPER + (loc & 7);
    return bm < nbm && bn < nbn;
  }
  // super-tile row r < nsn holds r full super-tiles and the diagonal one:
  // 64 r + 36 blocks, 32 r^2 + 4 r before it
  const int64_t tri_total = 32 * (int64_t)nsn * nsn + 4 * (int64_t)nsn;
  if (t < tri_total) {
    int64_t r = (int64_t)((sqrt(16.0 + 128.0 * (double)t) - 4.0) * (1.0 / 64.0));
    while (32 * r * r + 4 * r > t) --r;
    while (32 * (r + 1) * (r + 1) + 4 * (r + 1) <= t) ++r;
    const int64_t u = t - (32 * r * r + 4 * r);
    if (u < 64 * r) {
      const int loc = (int)(u & 63);
      bm = (int)r * UPD_SUPER + (loc >> 3);
      bn = (int)(u >> 6) * UPD_SUPER + (loc & 7);
    } else {
      const int v = (int)(u - 64 * r);               // 0 .. 35, row by row of the triangle
      int i = (int)((sqrtf(8.0f * (float)v + 1.0f) - 1.0f) * 0.5f);
      while (i * (i + 1) / 2 > v) --i;
      while ((i + 1) * (i + 2) / 2 <= v) ++i;
      bm = (int)r * UPD_SUPER + i;
      bn = (int)r * UPD_SUPER + (v - i * (i + 1) / 2);
    }
  } else {
    const int64_t u = t - tri_total;
    const int64_t row = u / (64 * (int64_t)nsn), w = u % (64 * (int64_t)nsn);
    const int loc = (int)(w & 63);
    bm = (nsn + (int)row) * UPD_SUPER + (loc >> 3);
    bn = (int)(w >> 6) * UPD_SUPER + (loc & 7);
  }
  return bm < nbm && bn < nbn && bn <= bm;
}

// Block of workgroup `id` in a launch that starts at the k0-th number of every
// XCD's range of `per` numbers.
__device__ __forceinline__ bool update_block_of(const bool lower, int64_t id, int64_t per, int64_t k0,
                                                int nbm, int nbn, int nsn, int swl, int& bm, int& bn) {
  const int xcd = (int)(id & 7);
  const int64_t k = k0 + (id >> 3);
  if (k >= per) return false;
  return update_block_of_number(lower, (int64_t)xcd * per + k, nbm, nbn, nsn, swl, bm, bn);
}

// Optional tail of a lower-triangular launch: the factorisation of the leaf that starts at
// C's top-left corner (w = 0: none), done by the workgroup that reduced that
// block.  Pointers as for leaf_factor_kernel.
template <typename T>
struct FusedLeaf {
  int w;
  T* dvec;
  T* dinv;
  T* linv;
  long long pivot0;
  DevFlags* flags;
  int spd;   // positive-definite form (see leaf_factor_body)
};

// TM = MFMA tiles per wavefront in each direction: 4 -> 128 x 128 block, 2 -> 64 x 64.
template <typename T, int TM>
struct UpdShape {
  using X = Mfma<T>;
  static constexpr int BK = X::BK;                                // K elements per slab: 128 bytes a row
  static constexpr int BM = 32 * TM, BN = 32 * TM;                // block of C per workgroup
  static constexpr int PIVOTS = 2 * (BM + BN) * BK;               // both operands, double buffered; then
  static constexpr int SLAB_ELEMS = PIVOTS + 4 * BK;              // the pivots of a slab (twice), likewise
  static constexpr int LDS_ELEMS = SLAB_ELEMS > FACTOR_LDS_ELEMS ? SLAB_ELEMS : FACTOR_LDS_ELEMS;
};

typedef __attribute__((address_space(1))) const void* upd_global_ptr;
typedef __attribute__((address_space(3))) void* upd_lds_ptr;

constexpr int DEVICE_SCOPE = 16;                      // the sc1 bit of a buffer or LDS-direct access
// A wavefront's SIZE bytes a lane from base + off (base the same in all lanes) straight to LDS, lane by lane
// from byte `at` on (the same in all lanes).  Written out because the compiler, told of the load, waits for
// it in front of the next read of anything in LDS; the caller counts these loads and waits for them by
// itself (s_waitcnt vmcnt).  `at` goes into m0 by the compiler's hand, which uses that register too: it knows
// what is in it, and the instruction in front of the load is the wait that a load has to keep behind a write of m0.
template <int SIZE, int SCOPE>
__device__ __forceinline__ void load_to_lds(const char* base, const unsigned off, const unsigned at) {
  const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)base);
  const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)((uintptr_t)base >> 32));
  const unsigned long long from = ((unsigned long long)hi << 32) | lo;
#define MDET_TO_LDS(WIDTH, BITS)                                                                        \
  asm volatile("s_nop 0\n\tglobal_load_lds_" WIDTH " %1, %2" BITS ::"{m0}"(at), "v"(off), "s"(from))
  static_assert((SIZE == 16 || SIZE == 4) && (SCOPE == 0 || SCOPE == DEVICE_SCOPE), "forms in use");
  if constexpr (SIZE == 16 && SCOPE == 0) MDET_TO_LDS("dwordx4", "");
  else if constexpr (SIZE == 16) MDET_TO_LDS("dwordx4", " sc1");
  else if constexpr (SCOPE == 0) MDET_TO_LDS("dword", "");
  else MDET_TO_LDS("dword", " sc1");
#undef MDET_TO_LDS
}

// One block (bm, bn) of C, by all threads of the workgroup (there are barriers inside); `lds` =
// LDS_ELEMS elements, which are not read any more when the last thread returns.
//
// Staging.  A slab is 128 bytes of K per operand row.  It goes from global memory
// straight into LDS (global_load_lds_dwordx4: every lane names its own 16 global
// bytes, and lane l's land at the wavefront's LDS base + 16 l), so it needs no
// staging registers, no LDS store instructions and no wait before the last strip of
// the slab before.  One such load fills 1 KB = 8 rows; a workgroup's four wavefronts issue
// BM/32 of them per operand and slab.  Rows are 128 bytes apart in LDS without
// padding; instead the eight 16-byte chunks of row r are stored in the order
// chunk ^ ((r >> 1) & 7), which a lane arranges by choosing what it loads.  The
// 16 lanes that fetch one MFMA operand (16 consecutive rows, same logical chunk)
// then hit 16 different bank groups.  The scaling by -d is applied to the A
// fragments as they come out of LDS (the same single rounding of a * (-d) as if
// it were applied on the way in).
//
// SCALED: C -= A B^T with operands that carry the diagonal scaling already (rows of
// the Cholesky factor, or a left operand L D): no pivots are read and no fragment is
// scaled.
// In both forms the accumulators start from -C, collect +A D B^T and are negated on
// the way out, which rounds exactly like C - A D B^T term by term and needs neither a
// negated operand nor a negated pivot.
template <typename T, int TM, bool SCALED = false>
__device__ __forceinline__ void schur_update_block(
    T* __restrict__ C, int64_t ldc, const T* __restrict__ A, int64_t lda,
    const T* __restrict__ B, int64_t ldb, const T* __restrict__ d, int M, int N, int K,
    const bool lower, const int bm, const int bn, const FusedLeaf<T>& fl, T* __restrict__ lds) {
  using X = Mfma<T>;
  using acc_t = typename X::acc_t;
  using vec_t = typename X::vec_t;
  constexpr int BK = X::BK, VEC = X::VEC;
  static_assert(BK * sizeof(T) == 128 && VEC * sizeof(T) == 16, "a slab row is eight 16-byte chunks");
  constexpr int WT = 16 * TM;                         // rows/cols of C per wavefront
  constexpr int BM = 2 * WT, BN = 2 * WT;             // block of C per workgroup
  constexpr int NV = BM / 32;                         // 1 KB loads per wavefront, operand and slab
  constexpr int KS = BK / 4;                          // MFMA k-steps per slab (= 2 chunks a lane)
  static_assert(KS == 2 * VEC, "a lane's share of a slab row is two chunks");

  T (*As)[BM * BK] = reinterpret_cast<T (*)[BM * BK]>(lds);
  T (*Bs)[BN * BK] = reinterpret_cast<T (*)[BN * BK]>(lds + 2 * BM * BK);

  const int row0 = bm * BM, col0 = bn * BN;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  // a wavefront whose 64 x 64 piece lies strictly above the diagonal has nothing to do
  const bool active = !(lower && (row0 + wm * WT + WT - 1 < col0 + wn * WT));

  // ---- global -> LDS staging --------------------------------------------
  // Load v of a wavefront covers rows 8 * (4 v + wave) .. + 7 of the block; lane l
  // brings physical chunk l & 7 of row l >> 3, i.e. logical chunk (l & 7) ^ swizzle.
  // Addresses: a base common to the workgroup (scalar registers; moves along K) plus
  // a 32-bit byte offset per lane and load that is fixed for the whole block (row
  // clamped at the ragged edge included).  The host checks that 128 rows of either
  // operand span less than 4 GiB.
  const char* Abase = reinterpret_cast<const char*>(A + (int64_t)row0 * lda);
  const char* Bbase = reinterpret_cast<const char*>(B + (int64_t)col0 * ldb);
  unsigned aoff[NV], boff[NV];
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    const int rt = 8 * (4 * v + wave) + (lane >> 3);          // row within the block
    const int chunk = (lane & 7) ^ ((rt >> 1) & 7);           // logical 16-byte chunk this lane brings
    int ar = rt; if (row0 + ar > M - 1) ar = M - 1 - row0;
    int br = rt; if (col0 + br > N - 1) br = N - 1 - col0;
    aoff[v] = (unsigned)(((int64_t)ar * lda + chunk * VEC) * (int64_t)sizeof(T));
    boff[v] = (unsigned)(((int64_t)br * ldb + chunk * VEC) * (int64_t)sizeof(T));
  }
  const unsigned lds0 = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)(upd_lds_ptr)lds);
  constexpr int LOADS = 2 * NV + (SCALED ? 0 : 1);            // a wavefront's, per slab
  auto gload = [&](const int part, const int kt, const int buf) {
    const unsigned kb = (unsigned)kt * (unsigned)(BK * sizeof(T));
    auto at = [&](const int e) { return lds0 + (unsigned)(e * (int)sizeof(T)); };
    if (part < 2 * NV) {
      const int v = part / 2, rows = 8 * (4 * v + wave);
      if (part % 2 == 0) load_to_lds<16, 0>(Abase + kb, aoff[v], at((buf * BM + rows) * BK));
      else load_to_lds<16, 0>(Bbase + kb, boff[v], at(((2 * BM + buf * BN) + rows) * BK));
    } else if constexpr (!SCALED) {
      // the slab's pivots, every wavefront the same, by both halves of it
      load_to_lds<4, 0>(reinterpret_cast<const char*>(d) + kb, 4u * (lane & 31), at(UpdShape<T, TM>::PIVOTS + buf * 2 * BK));
    }
  };
  // all of this wavefront's loads have landed, and behind the barrier those of all
  auto landed = [] {
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };

  const int nk = K / BK;            // (K is a multiple of 64: an even number of slabs, at least two)
  __builtin_assume(nk >= 64 / BK);
  auto first_slabs = [&] {
#pragma unroll
    for (int part = 0; part < LOADS; ++part) gload(part, 0, 0);
    landed();
#pragma unroll
    for (int part = 0; part < LOADS; ++part) gload(part, 1, 1);
  };

  // The workgroup that goes on to factor the leaf at the block's top left hands that part over in LDS
  // (the operand buffers are free behind a barrier) and leaves its write-back to the factorisation.
  const bool fuse = lower && fl.w > 0 && bm == 0 && bn == 0;
  const int wleaf = fuse ? fl.w : 0;
  const int r16 = lane & 15, g = lane >> 4;

  // A wavefront without a piece brings its share of the slabs and keeps the barriers company, on a way of its own
  // to the end of the block.  Where the two ways met in front of the stores, the accumulators were live on both, and in
  // fp64 88 registers' worth went to scratch memory (K = 128, M = N = 16384 lower: 0.91 ms, 0.83 without).
  if (!active) {
    first_slabs();
    for (int kt = 0; kt + 1 < nk; ++kt) {
      landed();
      if (kt + 2 < nk) {
#pragma unroll
        for (int part = 0; part < LOADS; ++part) gload(part, kt + 2, kt & 1);
      }
    }
    if (fuse) {
      __syncthreads();
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
          for (int j = 0; j < TM; ++j)
            leaf_tile_put<T>(lds, wm * WT + i * 16 + X::acc_row(lane, r), wn * WT + j * 16 + r16, wleaf, T(0));
    }
  } else {
    // The accumulators start from (minus) C and the products are added to them in
    // K order, so every entry is reduced term by term exactly as in the unblocked
    // recurrence a_ij - sum_k l_ik d_k l_jk; when the Schur complement is much
    // smaller than a_ij (low-rank Gram matrix plus a small shift) the late roundings
    // are then relative to the small running value, not to the full sum.
    acc_t acc[TM][TM];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TM; ++j) acc[i][j] = acc_t{0, 0, 0, 0};
#pragma unroll
    for (int i = 0; i < TM; ++i) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int grow = row0 + wm * WT + i * 16 + X::acc_row(lane, r);
        if (grow >= M) continue;
        const T* crow = C + (int64_t)grow * ldc;
#pragma unroll
        for (int j = 0; j < TM; ++j) {
          const int gcol = col0 + wn * WT + j * 16 + r16;
          if (gcol < N && (!lower || gcol <= grow)) acc[i][j][r] = crow[gcol];
        }
      }
    }

    // lane group g owns the KS consecutive k's [g*KS, (g+1)*KS) of a slab, i.e. its
    // logical chunks 2g and 2g+1; MFMA step s multiplies the s-th of them from every
    // group (any assignment of the slab's k's to steps is valid as long as A and B
    // use the same one).  Where those chunks sit in a row depends only on the lane
    // (rows 16 apart share the swizzle).
    const int sw = (r16 >> 1) & 7;
    const int c0 = ((2 * g) ^ sw) * VEC, c1 = ((2 * g + 1) ^ sw) * VEC;
    first_slabs();
    {
      // -C, in one go now that the loads have landed (negating each entry as it is
      // loaded would make every load wait for itself)
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TM; ++j)
#pragma unroll
          for (int r = 0; r < 4; ++r) acc[i][j][r] = -acc[i][j][r];
    }

    // Fragments are fetched one 16-row strip at a time, each fetch issued one stage ahead of its first
    // use, so that LDS latency hides behind the chain of MFMAs of the stage before.  Stage (i, j): all
    // KS products of accumulator (i, j) back to back.  In front of the last strip's products, when nothing
    // more is read of this slab, the wavefronts meet: the next slab has landed, whose first fragments
    // are fetched and scaled beside these products, and this one's place takes the slab after that,
    // one or two loads behind each group of products.
    T fa[2][KS], fb[TM][KS], nd[KS];
    auto fetch = [&](T (&f)[KS], const T* base) {
      const vec_t v0 = *reinterpret_cast<const vec_t*>(base + c0);
      const vec_t v1 = *reinterpret_cast<const vec_t*>(base + c1);
#pragma unroll
      for (int e = 0; e < VEC; ++e) { f[e] = v0[e]; f[VEC + e] = v1[e]; }
    };
    auto fetch_pivots = [&](const int buf) {
      if constexpr (!SCALED) {
#pragma unroll
        for (int h = 0; h < KS / VEC; ++h) {
          const vec_t v = *reinterpret_cast<const vec_t*>(lds + UpdShape<T, TM>::PIVOTS + buf * 2 * BK + g * KS + h * VEC);
#pragma unroll
          for (int e = 0; e < VEC; ++e) nd[h * VEC + e] = v[e];
        }
      }
    };
    auto scale = [&](T (&f)[KS]) {
      if constexpr (!SCALED) {
#pragma unroll
        for (int e = 0; e < KS; ++e) f[e] *= nd[e];
      }
    };
    auto rows_of = [&](const int buf) { return &As[buf][(wm * WT + r16) * BK]; };
    auto cols_of = [&](const int buf) { return &Bs[buf][(wn * WT + r16) * BK]; };
    // One slab.  MORE slabs follow: 2 and more, 1 or 0 (decided at compile time, so that the stages of a slab
    // form one straight run of instructions).
    auto slab = [&](const int kt, auto buf_tag, auto more_tag) {
      constexpr int BUF = decltype(buf_tag)::value, MORE = decltype(more_tag)::value;
      const T* as = rows_of(BUF);
      const T* bs = cols_of(BUF);
#pragma unroll
      for (int i = 0; i < TM; ++i) {
#pragma unroll
        for (int j = 0; j < TM; ++j) {
          if (i == 0 && j + 1 < TM) fetch(fb[j + 1], bs + (j + 1) * 16 * BK);
          if (j == TM - 1 && i + 1 < TM) fetch(fa[(i + 1) & 1], as + (i + 1) * 16 * BK);
          if (j == 0 && i > 0) scale(fa[i & 1]);
          if (i == TM - 1 && MORE > 0) {
            if (j == 0) {
              landed();
              fetch(fa[0], rows_of(BUF ^ 1));
              fetch_pivots(BUF ^ 1);
            }
            if (j == 1) fetch(fb[0], cols_of(BUF ^ 1));
            if (j == TM - 1) scale(fa[0]);
          }
          __builtin_amdgcn_sched_barrier(0);   // all of the above goes out before this stage's products
#pragma unroll
          for (int e = 0; e < KS; ++e) acc[i][j] = X::mfma(fa[i & 1][e], fb[j][e], acc[i][j]);
          __builtin_amdgcn_sched_barrier(0);
          if (i == TM - 1 && MORE > 1) {
#pragma unroll
            for (int part = 0; part < LOADS; ++part)
              if (part * TM / LOADS == j) gload(part, kt + 2, BUF);
          }
        }
      }
    };
    using Zero = std::integral_constant<int, 0>;
    using One = std::integral_constant<int, 1>;
    using Two = std::integral_constant<int, 2>;
    static_assert(TM % 2 == 0, "the last strip is in fa[1], the next slab's first goes to fa[0]");
    fetch(fa[0], rows_of(0));
    fetch(fb[0], cols_of(0));
    fetch_pivots(0);
    scale(fa[0]);
    int kt = 0;
    for (; kt + 2 < nk; kt += 2) {
      slab(kt, Zero{}, Two{});
      slab(kt + 1, One{}, Two{});
    }
    slab(kt, Zero{}, One{});
    slab(kt + 1, One{}, Zero{});

    // ---- epilogue: store the reduced block ----------------------------------
    // (The lane anew where registers are short: the compiler would keep what it knows of C's addresses and bounds
    // across K, and 40 to 50 of those registers are not there in fp64.  fp32 has them to spare, and is 2.5 % faster
    // so at K = 128.)
    int mine = lane;
    if constexpr (TM == 4 && sizeof(T) == 8) asm volatile("" : "+v"(mine));
    const int mine16 = mine & 15;
    if (fuse) {
      __syncthreads();
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
          for (int j = 0; j < TM; ++j)
            leaf_tile_put<T>(lds, wm * WT + i * 16 + X::acc_row(mine, r), wn * WT + j * 16 + mine16,
                             wleaf, -acc[i][j][r]);
    }
#pragma unroll
    for (int i = 0; i < TM; ++i) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int grow = row0 + wm * WT + i * 16 + X::acc_row(mine, r);
        if (grow >= M) continue;
        T* crow = C + (int64_t)grow * ldc;
#pragma unroll
        for (int j = 0; j < TM; ++j) {
          const int gcol = col0 + wn * WT + j * 16 + mine16;
          if (gcol < N && (!lower || gcol <= grow) && !(grow < wleaf && gcol < wleaf))
            crow[gcol] = -acc[i][j][r];
        }
      }
    }
  }
  if (fuse) {
    __syncthreads();
    leaf_factor_body<T, true>(C, ldc, fl.w, fl.dvec, fl.dinv, fl.linv, fl.pivot0, fl.flags, lds,
                              fl.spd);
  }
}

// One block per workgroup.
template <typename T, int TM, bool SCALED = false>
__device__ __forceinline__ void schur_update_body(
    T* __restrict__ C, int64_t ldc, const T* __restrict__ A, int64_t lda,
    const T* __restrict__ B, int64_t ldb, const T* __restrict__ d, int M, int N, int K,
    int nsn, int swl, const bool lower, int per, int k0, const FusedLeaf<T>& fl) {
  using Sh = UpdShape<T, TM>;
  __shared__ __attribute__((aligned(16))) T lds[Sh::LDS_ELEMS];
  int bm, bn;
  if (!update_block_of(lower, blockIdx.x, per, k0, (M + Sh::BM - 1) / Sh::BM,
                       (N + Sh::BN - 1) / Sh::BN, nsn, swl, bm, bn))
    return;
  schur_update_block<T, TM, SCALED>(C, ldc, A, lda, B, ldb, d, M, N, K, lower, bm, bn, fl, lds);
}

// Names for the same body: the update of the trailing matrix by a finished block
// column (the bulk of all work), and the updates inside a block column's own
// recursive factorisation (128- and 64-wide blocks; the small one spreads short
// launches over more compute units).  The latter sit on the chain of dependent
// launches and often share SIMDs with a workgroup of the former: they run at a
// raised wave priority.
template <typename T, bool SCALED = false>
__global__ __launch_bounds__(UPD_THREADS, 2) void trailing_update_kernel(
    T* __restrict__ C, int64_t ldc, const T* __restrict__ A, int64_t lda,
    const T* __restrict__ B, int64_t ldb, const T* __restrict__ d, int M, int N, int K, int nsn,
    int swl, int lower, int per, int k0) {
  const FusedLeaf<T> none{0, nullptr, nullptr, nullptr, 0, nullptr, 0};
  schur_update_body<T, 4, SCALED>(C, ldc, A, lda, B, ldb, d, M, N, K, nsn, swl, lower != 0, per, k0, none);
}
// The trailing update of a short block column: with 128 x 128 blocks it would have
// fewer workgroups than the device has compute units and last as long as one
// workgroup's walk along K; 64 x 64 blocks quarter that walk.
template <typename T, bool SCALED = false>
__global__ __launch_bounds__(UPD_THREADS) void trailing_update64_kernel(
    T* __restrict__ C, int64_t ldc, const T* __restrict__ A, int64_t lda,
    const T* __restrict__ B, int64_t ldb, const T* __restrict__ d, int M, int N, int K, int nsn,
    int swl, int lower, int per, int k0) {
  const FusedLeaf<T> none{0, nullptr, nullptr, nullptr, 0, nullptr, 0};
  schur_update_body<T, 2, SCALED>(C, ldc, A, lda, B, ldb, d, M, N, K, nsn, swl, lower != 0, per, k0, none);
}
template <typename T, bool SCALED = false>
__global__ __launch_bounds__(UPD_THREADS, 2) void panel_update_kernel(
    T* __restrict__ C, int64_t ldc, const T* __restrict__ A, int64_t lda,
    const T* __restrict__ B, int64_t ldb, const T* __restrict__ d, int M, int N, int K, int nsn,
    int swl, int lower, int per, int k0, FusedLeaf<T> fl) {
  __builtin_amdgcn_s_setprio(2);
  schur_update_body<T, 4, SCALED>(C, ldc, A, lda, B, ldb, d, M, N, K, nsn, swl, lower != 0, per, k0, fl);
}
template <typename T, bool SCALED = false>
__global__ __launch_bounds__(UPD_THREADS) void panel_update64_kernel(
    T* __restrict__ C, int64_t ldc, const T* __restrict__ A, int64_t lda,
    const T* __restrict__ B, int64_t ldb, const T* __restrict__ d, int M, int N, int K, int nsn,
    int swl, int lower, int per, int k0, FusedLeaf<T> fl) {
  __builtin_amdgcn_s_setprio(2);
  schur_update_body<T, 2, SCALED>(C, ldc, A, lda, B, ldb, d, M, N, K, nsn, swl, lower != 0, per, k0, fl);
}

// K = 64 exactly (the update of the columns right of a leaf by that leaf): both
// operands, the pivots and the C block are requested in one go and the whole
// product runs from LDS, so the launch costs one memory round trip instead of one
// per slab.  64 x 64 block of C per workgroup, 2 x 2 MFMA tiles per wavefront.
template <typename T, bool SCALED>
__device__ __forceinline__ void leaf_update_body(
    T* __restrict__ C, int64_t ldc, const T* __restrict__ A, int64_t lda,
    const T* __restrict__ B, int64_t ldb, const T* __restrict__ d, int M, int N, int nsn, int swl,
    int lower_, int per, const FusedLeaf<T>& fl) {
  __builtin_amdgcn_s_setprio(2);
  const bool lower = lower_ != 0;
  using X = Mfma<T>;
  using acc_t = typename X::acc_t;
  using vec_t = typename X::vec_t;
  constexpr int VEC = X::VEC, BK = X::BK, KS = BK / 4;
  constexpr int KT = 64;                                    // K
  constexpr int S = (KT * (int)sizeof(T) + 16) / (int)sizeof(T);   // padded LDS row, elements
  constexpr int VPR = KT / VEC;                             // 16-byte vectors per row
  constexpr int NV = VPR / 4;                               // per thread (4 threads per row)
  __shared__ __attribute__((aligned(16))) T lds[2 * 64 * S];
  static_assert(2 * 64 * S >= FACTOR_LDS_ELEMS, "the fused leaf needs the operand buffers");
  T* As = lds;
  T* Bs = lds + 64 * S;

  int bm, bn;
  if (!update_block_of(lower, blockIdx.x, per, 0, (M + 63) / 64, (N + 63) / 64, nsn, swl, bm, bn))
    return;
  const int row0 = bm * 64, col0 = bn * 64;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const int r16 = lane & 15, g = lane >> 4;
  const bool active = !(lower && (row0 + wm * 32 + 31 < col0 + wn * 32));

  const int srow = tid >> 2, sq = tid & 3;
  int ar = row0 + srow; if (ar > M - 1) ar = M - 1;
  int br = col0 + srow; if (br > N - 1) br = N - 1;
  const T* Ap = A + (int64_t)ar * lda + sq * NV * VEC;
  const T* Bp = B + (int64_t)br * ldb + sq * NV * VEC;
  const T* dp = d + sq * NV * VEC;
  vec_t ra[NV], rb[NV], rd[NV];
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    ra[v] = *reinterpret_cast<const vec_t*>(Ap + v * VEC);
    rb[v] = *reinterpret_cast<const vec_t*>(Bp + v * VEC);
    if constexpr (!SCALED) rd[v] = *reinterpret_cast<const vec_t*>(dp + v * VEC);
  }
  acc_t acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = acc_t{0, 0, 0, 0};
  if (active) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int grow = row0 + wm * 32 + i * 16 + X::acc_row(lane, r);
        if (grow >= M) continue;
        const T* crow = C + (int64_t)grow * ldc;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const int gcol = col0 + wn * 32 + j * 16 + r16;
          if (gcol < N && (!lower || gcol <= grow)) acc[i][j][r] = crow[gcol];
        }
      }
  }
  {
    T* as = &As[srow * S + sq * NV * VEC];
    T* bs = &Bs[srow * S + sq * NV * VEC];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      if constexpr (SCALED) *reinterpret_cast<vec_t*>(as + v * VEC) = -ra[v];
      else *reinterpret_cast<vec_t*>(as + v * VEC) = -(ra[v] * rd[v]);
      *reinterpret_cast<vec_t*>(bs + v * VEC) = rb[v];
    }
  }
  __syncthreads();
  if (active) {
#pragma unroll
    for (int slab = 0; slab < KT / BK; ++slab) {
      const T* as = &As[(wm * 32 + r16) * S + slab * BK + g * KS];
      const T* bs = &Bs[(wn * 32 + r16) * S + slab * BK + g * KS];
#pragma unroll
      for (int h = 0; h < KS / VEC; ++h) {
        vec_t fa[2], fb[2];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          fa[t] = *reinterpret_cast<const vec_t*>(as + t * 16 * S + h * VEC);
          fb[t] = *reinterpret_cast<const vec_t*>(bs + t * 16 * S + h * VEC);
        }
#pragma unroll
        for (int e = 0; e < VEC; ++e)
#pragma unroll
          for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) acc[i][j] = X::mfma(fa[i][e], fb[j][e], acc[i][j]);
      }
    }
  }
  // the workgroup that factors the leaf at C's top left hands it over in LDS
  const bool fuse = lower && fl.w > 0 && bm == 0 && bn == 0;
  const int wleaf = fuse ? fl.w : 0;
  if (fuse) {
    __syncthreads();   // everybody is done with the operands
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          leaf_tile_put<T>(lds, wm * 32 + i * 16 + X::acc_row(lane, r), wn * 32 + j * 16 + r16,
                           wleaf, acc[i][j][r]);
  }
  if (active) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int grow = row0 + wm * 32 + i * 16 + X::acc_row(lane, r);
        if (grow >= M) continue;
        T* crow = C + (int64_t)grow * ldc;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const int gcol = col0 + wn * 32 + j * 16 + r16;
          if (gcol < N && (!lower || gcol <= grow) && !(grow < wleaf && gcol < wleaf))
            crow[gcol] = acc[i][j][r];
        }
      }
  }
  if (fuse) {
    __syncthreads();
    leaf_factor_body<T, true>(C, ldc, fl.w, fl.dvec, fl.dinv, fl.linv, fl.pivot0, fl.flags, lds,
                              fl.spd);
  }
}

template <typename T, bool SCALED = false>
__global__ __launch_bounds__(UPD_THREADS) void leaf_update_kernel(
    T* __restrict__ C, int64_t ldc, const T* __restrict__ A, int64_t lda,
    const T* __restrict__ B, int64_t ldb, const T* __restrict__ d, int M, int N, int nsn, int swl,
    int lower_, int per, FusedLeaf<T> fl) {
  leaf_update_body<T, SCALED>(C, ldc, A, lda, B, ldb, d, M, N, nsn, swl, lower_, per, fl);
}

// General matrices (Sec. 2.2, Eq. 1: M = P L U): the matrix is two lower-triangular arrays
// qoff elements apart, the entries on and below the diagonal and the transposed entries
// above it.  The same update runs on both in one launch with two rows of workgroups
// (blockIdx.y): the first array takes A's rows there and B's rows in the second array,
// the second array the other way round.  C, A and B all point into the first array.
template <typename T>
struct GeneralOperands {
  T* C;
  const T* A;
  const T* B;
};
template <typename T>
__device__ __forceinline__ GeneralOperands<T> general_operands(T* C, const T* A, const T* B, int64_t qoff) {
  if (blockIdx.y != 0) return {C + qoff, A + qoff, B};
  return {C, A, B + qoff};
}
template <typename T>
__global__ __launch_bounds__(UPD_THREADS) void leaf_update_general_kernel(
    T* C, int64_t ldc, const T* A, int64_t lda, const T* B, int64_t ldb, const T* __restrict__ d,
    int M, int N, int nsn, int swl, int lower_, int per, int64_t qoff) {
  const GeneralOperands<T> o = general_operands<T>(C, A, B, qoff);
  const FusedLeaf<T> none{0, nullptr, nullptr, nullptr, 0, nullptr, 0};
  leaf_update_body<T, false>(o.C, ldc, o.A, lda, o.B, ldb, d, M, N, nsn, swl, lower_, per, none);
}
#define MDET_GENERAL_UPDATE_KERNEL(NAME, TM, OCC, PRIO)                                              \
  template <typename T>                                                                             \
  __global__ __launch_bounds__(UPD_THREADS, OCC) void NAME(                                         \
      T* C, int64_t ldc, const T* A, int64_t lda, const T* B, int64_t ldb, const T* __restrict__ d, \
      int M, int N, int K, int nsn, int swl, int lower, int per, int k0, int64_t qoff) {            \
    if (PRIO) __builtin_amdgcn_s_setprio(2);                                                        \
    const GeneralOperands<T> o = general_operands<T>(C, A, B, qoff);                                \
    const FusedLeaf<T> none{0, nullptr, nullptr, nullptr, 0, nullptr, 0};                           \
    schur_update_body<T, TM, false>(o.C, ldc, o.A, lda, o.B, ldb, d, M, N, K, nsn, swl, lower != 0, \
                                    per, k0, none);                                                 \
  }
MDET_GENERAL_UPDATE_KERNEL(trailing_update_general_kernel, 4, 2, 0)
MDET_GENERAL_UPDATE_KERNEL(trailing_update64_general_kernel, 2, 1, 0)
MDET_GENERAL_UPDATE_KERNEL(panel_update_general_kernel, 4, 2, 1)
MDET_GENERAL_UPDATE_KERNEL(panel_update64_general_kernel, 2, 1, 1)
#undef MDET_GENERAL_UPDATE_KERNEL

}  // namespace mdet
