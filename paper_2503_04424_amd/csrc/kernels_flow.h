// A block column factored by ONE launch: the leaves, the solves below them and the updates
// between them as tasks that wait for each other, instead of a chain of launches (leaf, solve,
// update, leaf, ...; Sec. 2.2).  Four forms: symmetric, positive definite (rows of the Cholesky factor,
// whose products need no pivots), symmetric with the pivots of a leaf taken from its whole
// diagonal, and general matrices as two lower-triangular arrays (GeneralOperands), every tile of
// which there is twice: its row tasks are two, its diagonal task has both.
//
// The column is cut into tiles of 64 x 64 entries, tile (i, j) in tile row i and tile column j.
// A workgroup takes the next task by number:
//   diagonal task j:  tiles (j, j-1) and (j, j) reduced by everything left of them; then, once
//                     leaf j-1 is there, tile (j, j-1) solved against it and its product taken off
//                     tile (j, j); then that factored;
//   row task (p, j):  the tiles of tile rows 2p and 2p + 1 in column j that no diagonal task has
//                     (rows from j + 2 on; from j + 1 in the last tile column) reduced; then, once
//                     leaf j is there, solved.
// Everything a task reads except its own tiles is final, and was written by tasks with lower
// numbers (tile column by tile column, the diagonal task first): whoever holds the lowest
// number that is not through can always go on, however many workgroups the device holds at a
// time, and a launch beside it may have the rest.  (A wait gives up after FLOW_PATIENCE all the
// same: the call then fails, it does not hang.)
//
// What bounds it, where a matrix is small: the chain of leaves.  From one leaf to the next are the
// hand-over through memory, the solve of the 64 rows below it, the product of these and the
// elimination (leaf_factor_body), 0.7 + 3.2 + 0.9 + 6.7 us in fp64; everything else runs beside
// that.  Between launches the same steps also wait for every workgroup of the launch before and
// for the next one to start, and the updates between the leaves lie on the chain as well.  Measured
// against the chain of launches, whole calls that keep their input: symmetric fp64 n = 512 229 -> 145 us,
// n = 1500 (positive definite) 603 -> 360, n = 5555 (positive definite) 3020 -> 1445, n = 8192 5873 -> 3550, fp32
// n = 10000 5940 -> 3380; block columns of 2048 beside a bulk update, n = 32768, 190.9 -> 174.6 ms; pivots from
// inside a leaf (23 us from leaf to leaf), n = 4096 3.04 -> 1.60 ms; general (25 us) n = 2900 2.27 -> 1.28, n = 8192 11.3 ->
// 6.9.
// Where a matrix is large: the
// matrix cores, in fp64 3.6 us for the 128 x 64 x 64 products of a row task of one column and 7.0 for
// 128 x 128 x 64 of two (positive-definite form 3.5 and 6.9; 3.4 and 6.8 at their peak; fp32 1.97 and 3.65 of 1.7
// and 3.4).  That takes a loop over the slabs of the operands with no jump in it but its own: with the loads
// under conditions and all issued at the start of a slab, where 40 of them keep the wavefronts from
// their products, it was 4.2 and 7.7 us (fp32 2.2 and 3.95; n = 8192 3.88 -> 3.55 ms, fp32 n = 10000 3.67 -> 3.38).
// One workgroup of eight wavefronts has a compute unit to itself (its LDS sees to that): two
// of four wavefronts each slow each other's leaves down, whose single wavefront then waits for
// the other's matrix instructions (n = 8192: 10.8 us a leaf instead of 6.7), and the sums of a
// diagonal task take twice as long.
//
// Memory.  The chiplets' L2 caches do not see each other's writes.  What one task hands to
// another is written through (stores at device scope) and complete before the tile row's
// counter says so; a task's own tiles are read past the caches; and finished tiles are read by
// ordinary loads: they cannot be in any cache from before, as long as no 128-byte line holds
// entries of two tiles.  Where the array's rows do not start on such lines (LINES = false) the
// operands are read past the caches as well.
//
// Order of the products of one entry: k rising in slabs of 128 bytes, inside a slab as
// schur_update_block takes them, each term (l d) l: what the update kernels do, so results do not
// depend on where a block column ends.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kernels_leaf.h"
#include "kernels_update.h"
#include "mfma.h"

namespace mdet {

constexpr int FLOW_WAVES = 8;
constexpr int FLOW_THREADS = 64 * FLOW_WAVES;
constexpr int FLOW_ROWS_HELD = SUB * FLOW_WAVES;      // rows of a row task: two tile rows
constexpr int FLOW_STAGES = 4;                        // slabs in LDS: one in use, the next there, two on their way
constexpr unsigned long long FLOW_PATIENCE = 60ull * 100000000ull;   // of the 100 MHz counter

// Words of device memory a launch needs, zero when it starts: the next task, failure, and per
// tile row the number of its finished tiles (of both arrays of a general matrix, one after the other).
struct FlowSync {
  unsigned ticket;
  unsigned failed;
  unsigned done[1];
};
enum FlowForm { FLOW_SYM, FLOW_SPD, FLOW_PIVOT, FLOW_GENERAL };
static inline int64_t flow_words(int64_t m, int arrays) { return 2 + arrays * ((m + LEAF - 1) / LEAF); }

// The tasks in their order, two tile columns j0 = 2 J and j1 = j0 + 1 at a time (ntr tile rows, ntp = ceil(ntr
// / 2) pairs of them, pair p tile rows 2 p and 2 p + 1; `arrays` tasks for each row task).  J < two:
//   diagonal task j0, row task (pair J + 1, column j0), diagonal task j1, row task (pair J + 1, column
//   j1), row tasks (pairs from J + 2 on, both columns);
// the others:
//   diagonal task j0, row tasks (pairs from J + 1 on, column j0), and the same for j1;
// and if the last tile column is a j0: its diagonal task, row tasks (pairs from J on, that column).
// Row tasks of both columns read their rows once for 128 columns and multiply twice as long between two
// barriers, but are twice as long: where few are left (flow_two) they would be waited for.  Those next
// to the diagonal, which the next diagonal tasks wait for, have one.
enum FlowKind { FLOW_DIAGONAL, FLOW_ROWS, FLOW_ROWS2, FLOW_NOTHING };
struct FlowOrder {
  int ntr, ntc, arrays, two;
  __host__ __device__ __forceinline__ int64_t pairs() const { return (ntr + 1) / 2; }
  // tasks in front of column pair J
  __host__ __device__ __forceinline__ int64_t before(int64_t J) const {
    const int64_t A = J < two ? J : two, ntp = pairs();
    const int64_t both = A * (2 + arrays * ntp) - arrays * (A * (A - 1) / 2);
    return both + (J - A) * (2 + 2 * arrays * (ntp - 1)) - arrays * (J * (J - 1) - A * (A - 1));
  }
  __host__ __device__ __forceinline__ int64_t tasks() const {
    const int64_t J = (ntc - 1) / 2;
    if (ntr == ntc) return before(J) + (ntc % 2 == 0 ? 2 : 1);
    return ntc % 2 == 0 ? before(J + 1) : before(J) + 1 + arrays * (pairs() - J);
  }
  // column (the first of two), array and pair of task t
  __host__ __device__ __forceinline__ FlowKind task(const int t, int& pair, int& array, int& j) const {
    const int last = (ntc - 1) / 2;
    int J = 0;
    for (int step = 1 << 24; step != 0; step >>= 1)
      if (J + step <= last && before(J + step) <= t) J += step;
    int r = (int)(t - before(J));
    j = 2 * J;
    pair = array = 0;
    if (r == 0) return FLOW_DIAGONAL;
    --r;
    const int below = arrays * (int)(pairs() - J - 1);   // row tasks of one column
    if (j + 1 >= ntc) {                                  // the last column, alone
      array = r % arrays;
      pair = J + r / arrays;
    } else if (J == last && ntr == ntc) {                // no rows below the last two
      ++j;
      return FLOW_DIAGONAL;
    } else {
      const int first = J < two ? arrays : below;        // row tasks of j0 in front of diagonal task j1
      if (r == first) {
        ++j;
        return FLOW_DIAGONAL;
      }
      if (r > 2 * first) {
        array = (r - 2 * first - 1) % arrays;
        pair = J + 2 + (r - 2 * first - 1) / arrays;
        return FLOW_ROWS2;
      }
      if (r > first) {
        ++j;
        r -= first + 1;
      }
      array = r % arrays;
      pair = J + 1 + r / arrays;
    }
    // (the last pair, of an odd number of rows, may have none for this column)
    const int top = j + 1 < ntc ? j + 2 : j + 1;
    return 2 * pair >= top || 2 * pair + 1 < ntr ? FLOW_ROWS : FLOW_NOTHING;
  }
};
// Column pairs with row tasks of both: symmetric matrices while 28 pairs of tile rows are left, general ones (two
// row tasks to each) while 4 are: their leaves take twice as long, so a longer task is waited for less.  Measured
// (in place, ms): symmetric, 16 20 28 36 pairs, fp64 n = 5555 1.54 1.47 1.52 1.54, n = 8192 3.51 3.59 3.42 3.45, n = 12300
// 11.1 11.2 11.0 11.1, fp32 n = 10000 3.28 3.31 3.26 3.31; general, 4 6 8 11 14 pairs, fp64 n = 2900 1.25 1.24 1.24 1.24
// 1.25, n = 5000 2.32 2.35 2.38 2.45 2.57, n = 8192 7.58 7.61 7.59 7.76 8.03, n = 16384 49.8 49.9 49.8 50.1 50.9, fp32 n =
// 8000 3.61 3.67 3.70 3.73 3.84.
static inline int flow_two(int64_t m, int64_t w, int arrays) {
  const int64_t pairs = (m + 2 * LEAF - 1) / (2 * LEAF), columns = (w + 2 * LEAF - 1) / (2 * LEAF);
  const int64_t two = pairs - (arrays == 2 ? 4 : 28);
  return (int)(two < 0 ? 0 : (two < columns ? two : columns));
}
static inline FlowOrder flow_order(int64_t m, int64_t w, int arrays, int two) {
  return FlowOrder{(int)((m + LEAF - 1) / LEAF), (int)((w + LEAF - 1) / LEAF), arrays, two};
}

// Four consecutive entries past the caches: `base` is the same in all lanes, `off` bytes from it.
typedef unsigned flow_u4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ __amdgpu_buffer_rsrc_t flow_rsrc(const void* base) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, 0xffffffffu, 0x00027000);
}
template <typename T>
__device__ __forceinline__ void flow_load4(__amdgpu_buffer_rsrc_t r, unsigned off, T (&v)[4]) {
#pragma unroll
  for (int h = 0; h < (int)sizeof(T) / 4; ++h) {
    const flow_u4 u = __builtin_amdgcn_raw_buffer_load_b128(r, (int)(off + 16 * h), 0, DEVICE_SCOPE);
    __builtin_memcpy(&v[h * (16 / (int)sizeof(T))], &u, 16);
  }
}
template <typename T, FlowForm FORM>
struct FlowShape {
  static constexpr int BK = Mfma<T>::BK;
  static constexpr int ARRAYS = FORM == FLOW_GENERAL ? 2 : 1;
  static constexpr int ROWS = FLOW_ROWS_HELD * BK, COLS = 2 * LEAF * BK;   // the slabs of the two operands
  static constexpr int STAGE = ROWS + COLS + 2 * BK;              // both, and the pivots (twice)
  static constexpr int SLABS = FLOW_STAGES * STAGE;
  // after the sums the same memory holds what a solve needs of its leaf (of both its halves, one after
  // the other), later the leaf that is factored, and behind that the solved tiles
  static constexpr int LEAF_ELEMS =
      FORM == FLOW_GENERAL ? LU_LDS_ELEMS : (FORM == FLOW_PIVOT ? PIVOT_LDS_ELEMS : FACTOR_LDS_ELEMS);
  static constexpr int TILES = ARRAYS * LEAF * LEAF;
  // 16 rows of a wavefront on their way out or into another order of columns: behind what a
  // solve needs in a row task; in a diagonal task behind the solved tile (general matrices: one wavefront's)
  static constexpr int ROW_STRIDE = LEAF + 16 / (int)sizeof(T);
  static constexpr int OUT = SUB * ROW_STRIDE;
  static constexpr int SOLVED = (LEAF_ELEMS + 3) / 4 * 4;
  static constexpr int ROW_OUT = LeafOperands<T>::ELEMS;
  static constexpr int DIAG_OUT = SOLVED + TILES;
  static constexpr int ROW_TILE = ROW_OUT + FLOW_WAVES * OUT;     // a tile as a column operand
  static constexpr int LATER_ROW = ROW_TILE + LEAF * LEAF;
  static constexpr int LATER_DIAG = DIAG_OUT + (FORM == FLOW_GENERAL ? 1 : 4) * OUT;
  static constexpr int LATER = LATER_ROW > LATER_DIAG ? LATER_ROW : LATER_DIAG;
  // (so much that a compute unit holds one workgroup)
  static constexpr int LDS_ELEMS = SLABS > LATER ? SLABS : LATER;
  static_assert(SOLVED >= ARRAYS * LeafOperands<T>::ELEMS && LDS_ELEMS * sizeof(T) + 64 <= 160 * 1024,
                "places in LDS");
};

// What all tasks of a launch share.  LINES: the arrays' rows start on 128-byte lines.
template <typename T, bool LINES>
struct FlowArgs {
  T* P;                 // the block column's diagonal entry
  int64_t ld;
  int m, w;             // rows, columns (w a multiple of LEAF, or m = w)
  T* dvec;              // its pivots and reciprocal pivots
  T* dinv;
  T* W;                 // its pivot-scaled copy (rows from wskip on), or null
  int64_t wld;
  int wskip;
  int64_t qoff;         // general matrices: elements to the array of the transposed upper triangle
  int* perm;            // with pivoting: the rows of each leaf in the order taken
  long long pivot0;
  DevFlags* flags;
  FlowSync* sync;
  FlowOrder order;
};

// A wavefront waits until the counter of every lane (`row` < 0: none) has reached `need`;
// the smallest of them, or -1 if the launch has failed.  A wait that gives up is reported as pivot
// 0, kind 8.
template <typename T, bool LINES>
__device__ __forceinline__ int flow_wait(const FlowArgs<T, LINES>& a, const int row, const int need) {
  unsigned long long since = 0;
  for (unsigned spins = 0;; ++spins) {
    const int v = row >= 0 ? (int)__hip_atomic_load(&a.sync->done[row], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                           : INT32_MAX;
    if (__ballot(v < need) == 0ull) {
      int least = __builtin_amdgcn_readlane(v, 0);
#pragma unroll
      for (int q = 1; q < 4; ++q) {
        const int o = __builtin_amdgcn_readlane(v, q);
        least = o < least ? o : least;
      }
      return least;
    }
    if ((spins & 255u) == 255u) {
      if (__hip_atomic_load(&a.sync->failed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0u) return -1;
      const unsigned long long now = __builtin_amdgcn_s_memrealtime();
      if (since == 0) since = now;
      if (now - since > FLOW_PATIENCE) {
        if ((threadIdx.x & 63) == 0) {
          __hip_atomic_store(&a.sync->failed, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          atomicMin(&a.flags->first_bad, 0ull);
          atomicExch(&a.flags->bad_kind, 8ull);
        }
        return -1;
      }
    }
    __builtin_amdgcn_s_sleep(1);
  }
}
// The same by the first wavefront for all threads of the workgroup, counters r0 to r3.
template <typename T, bool LINES>
__device__ __forceinline__ int flow_wait_all(const FlowArgs<T, LINES>& a, const int r0, const int r1, const int r2, const int r3,
                                             const int need, int* shared) {
  if (threadIdx.x < 64) {
    const int lane = threadIdx.x;
    const int v = flow_wait(a, lane == 0 ? r0 : (lane == 1 ? r1 : (lane == 2 ? r2 : (lane == 3 ? r3 : -1))), need);
    if (lane == 0) *shared = v;
  }
  __syncthreads();
  return __builtin_amdgcn_readfirstlane(*shared);
}
template <typename T, bool LINES>
__device__ __forceinline__ void flow_publish(const FlowArgs<T, LINES>& a, const int row, const int count) {
  __hip_atomic_store(&a.sync->done[row], (unsigned)count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The sub-blocks of tile (j, j), on and below its diagonal, of each wavefront of a diagonal task.  One
// array: wavefront 0 has (0, 0), which the elimination starts with, wavefronts 5 to 7 three each of
// the others (4, on the SIMD of wavefront 0, none).  Two arrays: wavefronts 0 to 3 share those of
// the first, the others those of the second.
struct FlowUnits {
  int count;
  int row[3], col[3];
  __device__ __forceinline__ FlowUnits(const int wave, const int arrays) {
    if (arrays == 1) {
      count = wave == 0 ? 1 : (wave >= 5 ? 3 : 0);
      row[0] = wave == 0 ? 0 : (wave == 5 ? 1 : (wave == 6 ? 2 : 3));
      col[0] = wave == 0 ? 0 : (wave == 5 ? 0 : 1);
      row[1] = wave == 5 ? 1 : (wave == 6 ? 2 : 3);
      col[1] = wave == 5 ? 1 : 2;
      row[2] = wave == 5 ? 2 : 3;
      col[2] = wave == 7 ? 3 : 0;
    } else {
      const int w = wave & 3;
      count = w >= 2 ? 3 : 2;
      row[0] = w;
      col[0] = 0;
      row[1] = w == 0 ? 3 : w;
      col[1] = w == 0 ? 3 : 1;
      row[2] = w;
      col[2] = 2;
    }
  }
};

// What a task reduces its tiles by: operand rows of two tile rows (of P or, general matrices, of the
// array behind it), in the order in which a slab holds them, and the counters that say how far
// they are.
template <typename T>
struct FlowOperands {
  const T* row[2];      // tile rows of the row operand; row[1] is not read by a diagonal task of one array
  const T* col[2];      // and of the column operand; the second one of KIND 2 and 3 only
  int left[2];          // rows of the matrix from row[v] on
  int counter[4];       // -1: none
};

// The sums of a task over the tiles k < nk left of it, slab by slab through LDS.
// Row task (KIND 0): x[t] += L_col D L_row^T (transposed: register r of a lane of row g of lanes is row
// l16 of this wavefront's 16 and column 16 t + 4 g + r, as in leaf_solve_body), for 16 of the 128 rows
// (`mine`: this wavefront has some).
// Diagonal task (KIND 1): the same by wavefronts 0 to 3 for the 64 rows of row[0], and s[u] += L_row D
// L_row^T of the FlowUnits.
// Diagonal task of a general matrix (KIND 2): the 64 rows of row[0] by col[0] and those of row[1] by
// col[1], and s[u] += row[0] D row[1]^T (wavefronts 0 to 3) and row[1] D row[0]^T (the others).
// Row task of two columns (KIND 3): as KIND 0, x[NSUB + t] by col[1].
// False if the launch has failed.
template <typename T, FlowForm FORM, int KIND, bool LINES>
__device__ __forceinline__ bool flow_accumulate(const FlowArgs<T, LINES>& a, const FlowOperands<T>& of, const int nk, const bool mine,
                                                typename Mfma<T>::acc_t (&x)[KIND == 3 ? 2 * NSUB : NSUB],
                                                typename Mfma<T>::acc_t (&s)[3], T* __restrict__ lds, int* shared) {
  using X = Mfma<T>;
  using vec_t = typename X::vec_t;
  using Sh = FlowShape<T, FORM>;
  constexpr bool SCALED = FORM == FLOW_SPD;
  constexpr int BK = Sh::BK, VEC = X::VEC, KS = BK / 4, PER_TILE = LEAF / BK;
  constexpr int RV = KIND == 1 ? 1 : 2, CV = KIND >= 2 ? 2 : 1;   // a wavefront's loads of each operand per slab
  constexpr int NT = KIND == 3 ? 2 * NSUB : NSUB;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, g = lane >> 4;

  // LDS-direct loads as in schur_update_block: 8 rows of 128 bytes each, the eight 16-byte chunks
  // of a row in the order chunk ^ ((row >> 1) & 7).  Load v brings rows 8 wave .. + 7 of tile row v.
  const int rt = 8 * wave + (lane >> 3);
  const int chunk = (lane & 7) ^ ((rt >> 1) & 7);
  unsigned roff[2], coff[2];
#pragma unroll
  for (int v = 0; v < RV; ++v) {
    const int rr = rt < of.left[v] ? rt : of.left[v] - 1;
    roff[v] = (unsigned)(((int64_t)rr * a.ld + chunk * VEC) * (int64_t)sizeof(T));
  }
#pragma unroll
  for (int v = 0; v < CV; ++v) coff[v] = (unsigned)(((int64_t)rt * a.ld + chunk * VEC) * (int64_t)sizeof(T));
  const unsigned lds0 = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)(upd_lds_ptr)lds);
  constexpr int LOADS = RV + CV + (SCALED ? 0 : 1);    // a wavefront's, per slab
  // (parts RV + CV - 1 bring the operands, the last one the pivots)
  auto request = [&](const int part, const int slab, const int stage) {
    constexpr int SCOPE = LINES ? 0 : DEVICE_SCOPE;
    const unsigned kb = (unsigned)slab * 128u;
    auto at = [&](const int e) { return lds0 + (unsigned)((stage * Sh::STAGE + e) * (int)sizeof(T)); };
    if (part < RV)
      load_to_lds<16, SCOPE>(reinterpret_cast<const char*>(of.row[part]) + kb, roff[part], at((part * LEAF + wave * 8) * BK));
    else if (part < RV + CV)
      load_to_lds<16, SCOPE>(reinterpret_cast<const char*>(of.col[part - RV]) + kb, coff[part - RV],
                             at(Sh::ROWS + ((part - RV) * LEAF + wave * 8) * BK));
    else if constexpr (!SCALED)       // the slab's pivots: 128 bytes, every wavefront the same, by both halves of it
      load_to_lds<4, 0>(reinterpret_cast<const char*>(a.dvec) + kb, 4u * (lane & 31), at(Sh::ROWS + Sh::COLS));
  };
  auto request_all = [&](const int slab, const int stage) {
#pragma unroll
    for (int part = 0; part < LOADS; ++part) request(part, slab, stage);
  };

  const int own_sw = (l16 >> 1) & 7;
  const int pc = solve_col<T>(l16), pc_sw = (pc >> 1) & 7;
  auto fetch = [&](T (&f)[KS], const T* from, const int sw) {
    const vec_t v0 = *reinterpret_cast<const vec_t*>(from + (((2 * g) ^ sw) * VEC));
    const vec_t v1 = *reinterpret_cast<const vec_t*>(from + (((2 * g + 1) ^ sw) * VEC));
#pragma unroll
    for (int e = 0; e < VEC; ++e) { f[e] = v0[e]; f[VEC + e] = v1[e]; }
  };
  const FlowUnits units(wave, KIND == 2 ? 2 : 1);
  const int half = KIND == 2 ? (wave >> 2) * LEAF * BK : 0;       // which of the column operands
  // The first operands of a slab, fetched while the slab before is multiplied.
  struct First { T row[KS], col[KS], d[KS]; } next;
  const bool sums = mine && (KIND != 1 || wave < 4);
  auto scale = [&](T (&f)[KS], const T (&d)[KS]) {
    if constexpr (!SCALED) {
#pragma unroll
      for (int e = 0; e < KS; ++e) f[e] *= d[e];
    }
  };
  auto prefetch = [&](const int stage) {
    const T* rs = lds + stage * Sh::STAGE;
    if constexpr (!SCALED) {
#pragma unroll
      for (int h = 0; h < KS / VEC; ++h) {
        const vec_t v = *reinterpret_cast<const vec_t*>(rs + Sh::ROWS + Sh::COLS + g * KS + h * VEC);
#pragma unroll
        for (int e = 0; e < VEC; ++e) next.d[h * VEC + e] = v[e];
      }
    }
    if (sums) {
      fetch(next.row, rs + (wave * SUB + l16) * BK, own_sw);
      fetch(next.col, rs + Sh::ROWS + half + pc * BK, pc_sw);
    }
  };
  // Operands are waited for in front of the fetch of the next ones and not, as the compiler
  // would have it where it has lost count, behind it.
  auto arrived = [&](T (&f)[KS]) {
#pragma unroll
    for (int e = 0; e < KS; ++e) asm volatile("" : "+v"(f[e]));
  };
  // the first operands are there: scaled in front of the barrier, not behind it
  auto ready = [&] {
    if constexpr (!SCALED) arrived(next.d);
    if (sums) {
      arrived(next.row);
      arrived(next.col);
      scale(next.row, next.d);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  // (`behind`: what is to go out while the first products run)
  auto multiply = [&](const int stage, const int following, auto behind) {
    const T* rs = lds + stage * Sh::STAGE;
    const T* cs = rs + Sh::ROWS + half;
    T nd[KS];
    if constexpr ((KIND == 1 || KIND == 2) && !SCALED) {
#pragma unroll
      for (int e = 0; e < KS; ++e) nd[e] = next.d[e];
    }
    if (sums) {
      T fr[KS], fc[NT][KS];
#pragma unroll
      for (int e = 0; e < KS; ++e) {
        fr[e] = next.row[e];
        fc[0][e] = next.col[e];
      }
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        if (t > 0) arrived(fc[t]);
        __builtin_amdgcn_sched_barrier(0);
        if (t + 1 < NT) fetch(fc[t + 1], cs + ((t + 1) * SUB + pc) * BK, pc_sw);
        if constexpr (KIND == 0 || KIND == 3) {
          if (t == NT - 2) prefetch(following);                        // (behind the last slab: whatever is there)
          if (t == NT - 1) ready();
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int e = 0; e < KS; ++e) x[t] = X::mfma(fc[t][e], fr[e], x[t]);
        __builtin_amdgcn_sched_barrier(0);
        // (one load at a time: 40 in a row take 640 of a slab's 4096 clocks)
#pragma unroll
        for (int part = t; part < LOADS; part += NT) behind(part);
      }
    } else {
#pragma unroll
      for (int part = 0; part < LOADS; ++part) behind(part);
    }
    if constexpr (KIND == 1 || KIND == 2) {
      const int mine0 = KIND == 2 ? (wave >> 2) * LEAF : 0, other0 = KIND == 2 ? LEAF - mine0 : 0;
#pragma unroll
      for (int u = 0; u < 3; ++u)
        if (u < units.count) {
          T fr[KS], fc[KS];
          fetch(fr, rs + (mine0 + units.row[u] * SUB + l16) * BK, own_sw);
          fetch(fc, rs + (other0 + units.col[u] * SUB + l16) * BK, own_sw);
          scale(fr, nd);
#pragma unroll
          for (int e = 0; e < KS; ++e) s[u] = X::mfma(fr[e], fc[e], s[u]);
        }
      prefetch(following);
    }
    if (KIND == 1 || KIND == 2 || !sums) ready();
  };
  // All but the newest slab's loads (`late`; or really all) of this wavefront have landed, and behind
  // the barrier those of all.
  auto landed = [](const bool late) {
    if (!late) asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    else if constexpr (LOADS == 5) asm volatile("s_waitcnt vmcnt(5) lgkmcnt(0)" ::: "memory");
    else if constexpr (LOADS == 4) asm volatile("s_waitcnt vmcnt(4) lgkmcnt(0)" ::: "memory");
    else if constexpr (LOADS == 3) asm volatile("s_waitcnt vmcnt(3) lgkmcnt(0)" ::: "memory");
    else asm volatile("s_waitcnt vmcnt(2) lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };

  int k = 0;
  while (k < nk) {
    int upto = flow_wait_all(a, of.counter[0], of.counter[1], of.counter[2], of.counter[3], k + 1, shared);
    if (upto < 0) return false;
    if (upto > nk) upto = nk;
    const int s0 = k * PER_TILE, s1 = upto * PER_TILE;
    request_all(s0, 0);
    request_all(s0 + 1, 1);                            // (a tile has at least two slabs)
    if (s0 + 2 < s1) request_all(s0 + 2, 2);
    landed(s0 + 2 < s1);
    prefetch(0);
    ready();
    // slab by slab; the next one has landed, for all wavefronts after the barrier, which also says
    // that all are through with the slab before this one: its place takes the third from here.
    // First without a condition on any of it
    int slab = s0;
    for (; slab + FLOW_STAGES + 2 < s1; slab += FLOW_STAGES) {
#pragma unroll
      for (int q = 0; q < FLOW_STAGES; ++q) {
        if (q > 0 || slab > s0) landed(true);
        multiply(q, (q + 1) % FLOW_STAGES,
                 [&](const int part) { request(part, slab + q + 3, (q + 3) % FLOW_STAGES); });
      }
    }
    for (; slab < s1; slab += FLOW_STAGES) {
#pragma unroll
      for (int q = 0; q < FLOW_STAGES; ++q) {
        if (PER_TILE % FLOW_STAGES != 0 && q % PER_TILE == 0 && slab + q >= s1) break;
        if (slab + q > s0) landed(slab + q + 2 < s1);
        multiply(q, (q + 1) % FLOW_STAGES, [&](const int part) {
          if (slab + q + 3 < s1) request(part, slab + q + 3, (q + 3) % FLOW_STAGES);
        });
      }
    }
    __syncthreads();                                   // the slabs' places are free
    k = upto;
  }
  return true;
}

// What the solve against a leaf needs, into LDS: as LeafOperands::stage, the inverses of the
// diagonal sub-blocks (wavefronts 0 to 3, one each) formed here from the leaf itself: the same
// operations in the same order as the elimination carries along, and no array of them for every
// leaf in flight.
template <typename T>
struct FlowStage {
  using L = LeafOperands<T>;
  static constexpr int LOW = L::COUNT - NSUB, VEC = L::VEC;
  const int lane, c, g, row;
  __device__ __forceinline__ FlowStage(const int lane_) : lane(lane_), c(lane_ & 15), g(lane_ >> 4), row(solve_col<T>(lane_ & 15)) {}
  // row c of diagonal sub-block b
  __device__ __forceinline__ void load_diagonal(const T* __restrict__ leaf, const int64_t ld, const int b, T (&nl)[SUB]) const {
    const T* mine = leaf + (int64_t)(b * SUB + c) * ld + b * SUB;
#pragma unroll
    for (int k = 0; k < SUB; k += 4) {
      T f[4];
      load4(mine + k, f);
#pragma unroll
      for (int e = 0; e < 4; ++e) nl[k + e] = f[e];
    }
  }
  // its inverse to LDS
  __device__ __forceinline__ void put_inverse(const L& ops, const int b, T (&nl)[SUB]) const {
    T inv[4];
#pragma unroll
    for (int k = 0; k < SUB; ++k) nl[k] = c > k ? -nl[k] : T(0);
#pragma unroll
    for (int s = 0; s < 4; ++s) inv[s] = Mfma<T>::acc_row(lane, s) == c ? T(1) : T(0);
    invert16_rows(inv, nl);
    // entry (c, k) belongs to the lane whose operand row is c (solve_col is its own inverse)
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int k = Mfma<T>::acc_row(lane, s), e = k & 3;
      ops.lds[(((LOW + b) * (4 / VEC) + e / VEC) * 64 + (k >> 2) * 16 + row) * VEC + e % VEC] = inv[s];
    }
  }
  // this lane's share of the q-th sub-block below the diagonal, and minus it to LDS
  __device__ __forceinline__ void load_lower(const T* __restrict__ leaf, const int64_t ld, const int q, T (&v)[4]) const {
    const int b = q < 1 ? 1 : (q < 3 ? 2 : 3);
    load4(leaf + (int64_t)(b * SUB + row) * ld + (q - L::lower(b, 0)) * SUB + 4 * g, v);
  }
  __device__ __forceinline__ void put_lower(const L& ops, const int q, const T (&v)[4]) const {
#pragma unroll
    for (int h = 0; h < 4 / VEC; ++h) {
      typename L::vec_t o;
#pragma unroll
      for (int e = 0; e < VEC; ++e) o[e] = -v[VEC * h + e];
      *ops.at(q, h, lane) = o;
    }
  }
};
template <typename T>
__device__ __forceinline__ void flow_stage_leaf(const LeafOperands<T>& ops, const T* __restrict__ leaf, const int64_t ld,
                                                const int wave, const int lane) {
  using St = FlowStage<T>;
  const St st(lane);
  if (wave < 4) {
    T nl[SUB];
    st.load_diagonal(leaf, ld, wave, nl);
    st.put_inverse(ops, wave, nl);
  } else {
    T v[2][4];
#pragma unroll
    for (int k = 0; k < 2; ++k)
      if (4 * k + wave - 4 < St::LOW) st.load_lower(leaf, ld, 4 * k + wave - 4, v[k]);
#pragma unroll
    for (int k = 0; k < 2; ++k)
      if (4 * k + wave - 4 < St::LOW) st.put_lower(ops, 4 * k + wave - 4, v[k]);
  }
}
// The same for a general matrix' L and U^T at once: the inverses by wavefronts 0 to 3, two each, the others by
// those that have columns to reorder besides.
template <typename T>
__device__ __forceinline__ void flow_stage_both(const LeafOperands<T>& opsL, const LeafOperands<T>& opsU,
                                                const T* __restrict__ L, const T* __restrict__ U, const int64_t ld,
                                                const int wave, const int lane) {
  using St = FlowStage<T>;
  static_assert(2 * St::LOW == 12, "three sub-blocks to a wavefront");
  const St st(lane);
  if (wave < 4) {
    T nl[2][SUB];
    st.load_diagonal(L, ld, wave, nl[0]);
    st.load_diagonal(U, ld, wave, nl[1]);
    st.put_inverse(opsL, wave, nl[0]);
    st.put_inverse(opsU, wave, nl[1]);
  } else {
    T v[3][4];
    auto of = [&](const int k) { return 4 * k + wave - 4; };
#pragma unroll
    for (int k = 0; k < 3; ++k) st.load_lower(of(k) < 6 ? L : U, ld, of(k) < 6 ? of(k) : of(k) - 6, v[k]);
#pragma unroll
    for (int k = 0; k < 3; ++k) st.put_lower(of(k) < 6 ? opsL : opsU, of(k) < 6 ? of(k) : of(k) - 6, v[k]);
  }
}

// 16 solved, divided rows of `array` from r16 on (this lane's share of them, columns of tile column col)
// to memory and, scaled by the pivots, to the copy.  The first through LDS (`out`, this wavefront's), so
// that a store writes whole rows: in 16-byte pieces as the lanes hold them a row task's 64 KB
// took 2.9 us to arrive.
template <typename T, bool LINES>
__device__ __forceinline__ void flow_store_rows(const FlowArgs<T, LINES>& a, T* array, const int64_t r16, const int col,
                                                const T (&v)[NSUB][4], T* __restrict__ out, const int lane) {
  using vec_t = typename Mfma<T>::vec_t;
  constexpr int VEC = Mfma<T>::VEC, STRIDE = FlowShape<T, FLOW_SYM>::ROW_STRIDE;
  constexpr int PIECES = LEAF / VEC, ROWS = 64 / PIECES;         // 16-byte pieces of a row, rows of a store
  const int l16 = lane & 15, g = lane >> 4;
#pragma unroll
  for (int b = 0; b < NSUB; ++b)
#pragma unroll
    for (int h = 0; h < 4 / VEC; ++h) {
      vec_t o;
#pragma unroll
      for (int e = 0; e < VEC; ++e) o[e] = v[b][VEC * h + e];
      *reinterpret_cast<vec_t*>(out + l16 * STRIDE + b * SUB + 4 * g + VEC * h) = o;
    }
  const __amdgpu_buffer_rsrc_t to = flow_rsrc(array + r16 * a.ld + (int64_t)col * LEAF);
  const int r0 = lane / PIECES, c = (lane % PIECES) * VEC;
#pragma unroll
  for (int q = 0; q < SUB / ROWS; ++q) {
    const int r = q * ROWS + r0;
    const vec_t o = *reinterpret_cast<const vec_t*>(out + r * STRIDE + c);
    flow_u4 u;
    __builtin_memcpy(&u, &o, 16);
    if (r16 + r < a.m)
      __builtin_amdgcn_raw_buffer_store_b128(u, to, (int)(unsigned)(((int64_t)r * a.ld + c) * (int64_t)sizeof(T)), 0,
                                             DEVICE_SCOPE);
  }
  if (a.W != nullptr && r16 + l16 < a.m && r16 + l16 >= a.wskip) {
    T d[NSUB][4];
    load_row((const T*)(a.dvec + (int64_t)col * LEAF), g, LEAF, d);
#pragma unroll
    for (int b = 0; b < NSUB; ++b)
#pragma unroll
      for (int e = 0; e < 4; ++e) d[b][e] *= v[b][e];
    store_row(a.W + (r16 + l16) * a.wld + (int64_t)col * LEAF, g, LEAF, d);
  }
}

// 16 rows of `array` in tile column col, negated, as flow_accumulate collects them.
template <typename T, bool LINES>
__device__ __forceinline__ void flow_load_rows(const FlowArgs<T, LINES>& a, const T* array, const int64_t r16, const int col,
                                               typename Mfma<T>::acc_t* x, const int lane) {
  const int l16 = lane & 15, g = lane >> 4;
  const __amdgpu_buffer_rsrc_t from = flow_rsrc(array + r16 * a.ld + (int64_t)col * LEAF);
  const unsigned off = (unsigned)(((int64_t)l16 * a.ld + 4 * g) * (int64_t)sizeof(T));
  T v[NSUB][4];
#pragma unroll
  for (int b = 0; b < NSUB; ++b)
#pragma unroll
    for (int e = 0; e < 4; ++e) v[b][e] = T(0);
  if (r16 + l16 < a.m) {
#pragma unroll
    for (int b = 0; b < NSUB; ++b) flow_load4(from, off + (unsigned)(b * SUB * sizeof(T)), v[b]);
  }
#pragma unroll
  for (int b = 0; b < NSUB; ++b)
#pragma unroll
    for (int e = 0; e < 4; ++e) x[b][e] = -v[b][e];
}

// Solve of this wavefront's 16 rows against the staged leaf, its operands fetched ahead: x from
// minus the reduced rows to the solved ones, undivided.  (The operations of LeafOperands::solve.)
template <typename T>
__device__ __forceinline__ void flow_solve(const LeafOperands<T>& ops, typename Mfma<T>::acc_t* x, const int lane) {
  using X = Mfma<T>;
  using L = LeafOperands<T>;
  using acc_t = typename X::acc_t;
  constexpr int LOW = L::COUNT - NSUB;
  T op[L::COUNT][4];
#pragma unroll
  for (int b = 0; b < NSUB; ++b) {
#pragma unroll
    for (int p = 0; p < b; ++p) ops.fetch(L::lower(b, p), lane, op[L::lower(b, p)]);
    ops.fetch(LOW + b, lane, op[LOW + b]);
  }
#pragma unroll
  for (int b = 0; b < NSUB; ++b) x[b] = -x[b];
#pragma unroll
  for (int b = 0; b < NSUB; ++b) {
#pragma unroll
    for (int p = 0; p < b; ++p)
#pragma unroll
      for (int s = 0; s < 4; ++s) x[b] = X::mfma(op[L::lower(b, p)][s], x[p][s], x[b]);
    acc_t wb = acc_t{0, 0, 0, 0};
#pragma unroll
    for (int s = 0; s < 4; ++s) wb = X::mfma(op[LOW + b][s], x[b][s], wb);
    x[b] = wb;
  }
}

// The columns of this wavefront's 16 rows into the order in which the leaf's rows were taken, through
// `out` (this wavefront's).  The order is asked for (ahead of the leaf) and used in two steps.
struct FlowGather {
  int from[NSUB][4];
  __device__ __forceinline__ void load(const int* __restrict__ perm, const int lane) {
    const int g = lane >> 4;
#pragma unroll
    for (int b = 0; b < NSUB; ++b) load4(perm + b * SUB + 4 * g, from[b]);
  }
  template <typename T>
  __device__ __forceinline__ void apply(const long long first, typename Mfma<T>::acc_t* x, T* __restrict__ out, const int lane) const {
    constexpr int STRIDE = FlowShape<T, FLOW_SYM>::ROW_STRIDE;
    const int l16 = lane & 15, g = lane >> 4;
#pragma unroll
    for (int b = 0; b < NSUB; ++b)
#pragma unroll
      for (int e = 0; e < 4; ++e) out[l16 * STRIDE + b * SUB + 4 * g + e] = x[b][e];
#pragma unroll
    for (int b = 0; b < NSUB; ++b)
#pragma unroll
      for (int e = 0; e < 4; ++e) x[b][e] = out[l16 * STRIDE + (from[b][e] - (int)first)];
  }
};

template <typename T, FlowForm FORM, bool LINES>
__device__ __forceinline__ void flow_row_task(const FlowArgs<T, LINES>& a, const int pair, const int array, const int j,
                                              T* __restrict__ lds, int* shared) {
  using acc_t = typename Mfma<T>::acc_t;
  using Sh = FlowShape<T, FORM>;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // of the pair's two tile rows those that this task has; the other one, whose entries left of
  // column j need not be final, is not read at all
  const int first = j + 1 < a.order.ntc ? j + 2 : j + 1;
  const bool low = 2 * pair >= first, high = 2 * pair + 1 < a.order.ntr;
  const int rt0 = low ? 2 * pair : 2 * pair + 1, rt1 = high ? 2 * pair + 1 : 2 * pair;
  const int64_t r16 = (int64_t)pair * FLOW_ROWS_HELD + wave * SUB;
  const bool mine = (wave < 4 ? low : high) && r16 < a.m;
  // general matrices: the rows of one array by those of the other, and solved against the leaf there
  T* const rows = a.P + (FORM == FLOW_GENERAL && array != 0 ? a.qoff : 0);
  T* const cols = a.P + (FORM == FLOW_GENERAL && array == 0 ? a.qoff : 0);
  const int mine0 = FORM == FLOW_GENERAL ? array * a.order.ntr : 0, other0 = FORM == FLOW_GENERAL ? (1 - array) * a.order.ntr : 0;
  FlowOperands<T> of;
  of.row[0] = rows + (int64_t)rt0 * LEAF * a.ld;
  of.row[1] = rows + (int64_t)rt1 * LEAF * a.ld;
  of.left[0] = a.m - rt0 * LEAF;
  of.left[1] = a.m - rt1 * LEAF;
  of.col[0] = of.col[1] = cols + (int64_t)j * LEAF * a.ld;
  of.counter[0] = mine0 + rt0;
  of.counter[1] = mine0 + rt1;
  of.counter[2] = other0 + j;
  of.counter[3] = -1;
  acc_t x[NSUB], none[3];
#pragma unroll
  for (int b = 0; b < NSUB; ++b) x[b] = acc_t{0, 0, 0, 0};
  if (mine) flow_load_rows(a, (const T*)rows, r16, j, x, lane);
  if (!flow_accumulate<T, FORM, 0>(a, of, j, mine, x, none, lds, shared)) return;
  if (flow_wait_all(a, j, -1, -1, -1, j + 1, shared) < 0) return;
  const LeafOperands<T> ops{lds};
  const bool gather = FORM == FLOW_PIVOT || (FORM == FLOW_GENERAL && array != 0);
  FlowGather order;
  if (gather) order.load((const int*)(a.perm + (int64_t)j * LEAF), lane);
  flow_stage_leaf(ops, (const T*)(cols + (int64_t)j * LEAF * (a.ld + 1)), a.ld, wave, lane);
  T rinv[NSUB][4];
  load_row((const T*)(a.dinv + (int64_t)j * LEAF), lane >> 4, LEAF, rinv);
  T* const out = lds + Sh::ROW_OUT + wave * Sh::OUT;
  if (gather && mine) order.apply(a.pivot0 + (long long)j * LEAF, x, out, lane);
  __syncthreads();
  if (mine) {
    flow_solve(ops, x, lane);
    T v[NSUB][4];
#pragma unroll
    for (int b = 0; b < NSUB; ++b)
#pragma unroll
      for (int e = 0; e < 4; ++e) v[b][e] = x[b][e] * rinv[b][e];
    flow_store_rows(a, rows, r16, j, v, out, lane);
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (tid == 0) {
    flow_publish(a, mine0 + rt0, j + 1);
    if (rt1 != rt0) flow_publish(a, mine0 + rt1, j + 1);
  }
}

// A row task of columns j and j + 1, the tile rows of the pair whole and far from the diagonal: behind the
// solve of the first column's tiles their products with tile (j + 1, j) come off the second's.
template <typename T, FlowForm FORM, bool LINES>
__device__ __forceinline__ void flow_row2_task(const FlowArgs<T, LINES>& a, const int pair, const int array, const int j,
                                               T* __restrict__ lds, int* shared) {
  using X = Mfma<T>;
  using acc_t = typename X::acc_t;
  using vec_t = typename X::vec_t;
  using Sh = FlowShape<T, FORM>;
  constexpr bool SCALED = FORM == FLOW_SPD;
  constexpr int BK = X::BK, VEC = X::VEC, KS = BK / 4;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, g = lane >> 4;
  const int rt0 = 2 * pair, rt1 = rt0 + 1 < a.order.ntr ? rt0 + 1 : rt0;
  const int64_t r16 = (int64_t)pair * FLOW_ROWS_HELD + wave * SUB;
  const bool mine = r16 < a.m;
  T* const rows = a.P + (FORM == FLOW_GENERAL && array != 0 ? a.qoff : 0);
  T* const cols = a.P + (FORM == FLOW_GENERAL && array == 0 ? a.qoff : 0);
  const int mine0 = FORM == FLOW_GENERAL ? array * a.order.ntr : 0, other0 = FORM == FLOW_GENERAL ? (1 - array) * a.order.ntr : 0;
  const bool gather = FORM == FLOW_PIVOT || (FORM == FLOW_GENERAL && array != 0);
  FlowOperands<T> of;
  of.row[0] = rows + (int64_t)rt0 * LEAF * a.ld;
  of.row[1] = rows + (int64_t)rt1 * LEAF * a.ld;
  of.left[0] = a.m - rt0 * LEAF;
  of.left[1] = a.m - rt1 * LEAF;
  of.col[0] = cols + (int64_t)j * LEAF * a.ld;
  of.col[1] = of.col[0] + LEAF * a.ld;
  of.counter[0] = mine0 + rt0;
  of.counter[1] = mine0 + rt1;
  of.counter[2] = other0 + j;
  of.counter[3] = other0 + j + 1;
  acc_t x[2 * NSUB], none[3];
#pragma unroll
  for (int b = 0; b < 2 * NSUB; ++b) x[b] = acc_t{0, 0, 0, 0};
  if (mine) {
    flow_load_rows(a, (const T*)rows, r16, j, x, lane);
    flow_load_rows(a, (const T*)rows, r16, j + 1, x + NSUB, lane);
  }
  if (!flow_accumulate<T, FORM, 3>(a, of, j, mine, x, none, lds, shared)) return;
  const LeafOperands<T> ops{lds};
  T* const out = lds + Sh::ROW_OUT + wave * Sh::OUT;
  T* const tile = lds + Sh::ROW_TILE;
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    if (flow_wait_all(a, j + c, -1, -1, -1, j + c + 1, shared) < 0) return;
    FlowGather order;
    if (gather) order.load((const int*)(a.perm + (int64_t)(j + c) * LEAF), lane);
    flow_stage_leaf(ops, (const T*)(cols + (int64_t)(j + c) * LEAF * (a.ld + 1)), a.ld, wave, lane);
    T rinv[NSUB][4];
    load_row((const T*)(a.dinv + (int64_t)(j + c) * LEAF), g, LEAF, rinv);
    if (gather && mine) order.apply(a.pivot0 + (long long)(j + c) * LEAF, x + c * NSUB, out, lane);
    __syncthreads();
    if (mine) {
      flow_solve(ops, x + c * NSUB, lane);
      T v[NSUB][4];
#pragma unroll
      for (int b = 0; b < NSUB; ++b)
#pragma unroll
        for (int e = 0; e < 4; ++e) v[b][e] = x[c * NSUB + b][e] * rinv[b][e];
      flow_store_rows(a, rows, r16, j + c, v, out, lane);
    }
    if (c == 0) {
      // tile (j + 1, j) as slabs of a column operand
      if (flow_wait_all(a, other0 + j + 1, -1, -1, -1, j + 1, shared) < 0) return;
      const int rt = 8 * wave + (lane >> 3);
      const int chunk = (lane & 7) ^ ((rt >> 1) & 7);
      const T* from = of.col[1] + (int64_t)rt * a.ld + (int64_t)j * LEAF + chunk * VEC;
#pragma unroll
      for (int p = 0; p < LEAF / BK; ++p) {
        __builtin_amdgcn_global_load_lds((upd_global_ptr)(from + p * BK), (upd_lds_ptr)(tile + (p * LEAF + wave * 8) * BK), 16,
                                         0, LINES ? 0 : DEVICE_SCOPE);
      }
      T d[NSUB][4];                    // the pivots in the order of the product
      if constexpr (!SCALED) {
#pragma unroll
        for (int q = 0; q < NSUB; ++q)
          load4((const T*)(a.dvec + (int64_t)j * LEAF + q / (KS / 4) * BK + g * KS + q % (KS / 4) * 4), d[q]);
      }
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");           // the solved rows are out, the tile is in
      __syncthreads();
      if (tid == 0) {
        flow_publish(a, mine0 + rt0, j + 1);
        if (rt1 != rt0) flow_publish(a, mine0 + rt1, j + 1);
      }
      if (mine) {
        const int pc = solve_col<T>(l16), sw = (pc >> 1) & 7;
#pragma unroll
        for (int p = 0; p < LEAF / BK; ++p) {
          T fr[KS], fc[NSUB][KS];
#pragma unroll
          for (int h = 0; h < KS / VEC; ++h) {
            const vec_t v = *reinterpret_cast<const vec_t*>(out + l16 * Sh::ROW_STRIDE + p * BK + g * KS + h * VEC);
#pragma unroll
            for (int e = 0; e < VEC; ++e) fr[h * VEC + e] = v[e];
          }
#pragma unroll
          for (int t = 0; t < NSUB; ++t) {
            const T* at = tile + (p * LEAF + t * SUB + pc) * BK;
            const vec_t v0 = *reinterpret_cast<const vec_t*>(at + (((2 * g) ^ sw) * VEC));
            const vec_t v1 = *reinterpret_cast<const vec_t*>(at + (((2 * g + 1) ^ sw) * VEC));
#pragma unroll
            for (int e = 0; e < VEC; ++e) { fc[t][e] = v0[e]; fc[t][VEC + e] = v1[e]; }
          }
          if constexpr (!SCALED) {
#pragma unroll
            for (int e = 0; e < KS; ++e) fr[e] *= d[p * (KS / 4) + e / 4][e % 4];
          }
#pragma unroll
          for (int t = 0; t < NSUB; ++t)
#pragma unroll
            for (int e = 0; e < KS; ++e) x[NSUB + t] = X::mfma(fc[t][e], fr[e], x[NSUB + t]);
        }
      }
    }
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (tid == 0) {
    flow_publish(a, mine0 + rt0, j + 2);
    if (rt1 != rt0) flow_publish(a, mine0 + rt1, j + 2);
  }
}

// Place in LDS of entries [VEC h, VEC h + VEC) of lane l's four of sub-block (q, b) of a solved tile.
template <typename T>
__device__ __forceinline__ typename Mfma<T>::vec_t* flow_solved_at(T* solved, const int q, const int b, const int h,
                                                                   const int l) {
  constexpr int VEC = Mfma<T>::VEC;
  return reinterpret_cast<typename Mfma<T>::vec_t*>(solved + (((q * NSUB + b) * (4 / VEC) + h) * 64 + l) * VEC);
}
template <typename T>
__device__ __forceinline__ void flow_solved_fetch(T* solved, const int q, const int b, const int l, T (&f)[4]) {
  constexpr int VEC = Mfma<T>::VEC;
#pragma unroll
  for (int h = 0; h < 4 / VEC; ++h) {
    const typename Mfma<T>::vec_t o = *flow_solved_at(solved, q, b, h, l);
#pragma unroll
    for (int e = 0; e < VEC; ++e) f[VEC * h + e] = o[e];
  }
}
// This wavefront's solved rows, divided (v), to the others.
template <typename T>
__device__ __forceinline__ void flow_solved_put(T* solved, const int q, const typename Mfma<T>::acc_t (&x)[NSUB],
                                                const T (&rinv)[NSUB][4], T (&v)[NSUB][4], const int lane) {
  constexpr int VEC = Mfma<T>::VEC;
#pragma unroll
  for (int b = 0; b < NSUB; ++b)
#pragma unroll
    for (int h = 0; h < 4 / VEC; ++h) {
      typename Mfma<T>::vec_t o;
#pragma unroll
      for (int e = 0; e < VEC; ++e) o[e] = v[b][VEC * h + e] = x[b][VEC * h + e] * rinv[b][VEC * h + e];
      *flow_solved_at(solved, q, b, h, lane) = o;
    }
}
// Operands of slab p (KS consecutive columns of each BK to a row of lanes) from 16 solved rows.
template <typename T, int KS>
__device__ __forceinline__ void flow_solved_slab(T* solved, const int q, const int p, const int l16, const int g, T (&f)[KS]) {
#pragma unroll
  for (int h = 0; h < KS / 4; ++h) {
    // columns c .. c + 3 are with sub-block c / 16 and row of lanes c / 4 % 4
    const int c = p * 4 * KS + g * KS + 4 * h;
    T v[4];
    flow_solved_fetch(solved, q, c / SUB, (c / 4 % 4) * 16 + l16, v);
#pragma unroll
    for (int e = 0; e < 4; ++e) f[4 * h + e] = v[e];
  }
}

// The symmetric forms.
template <typename T, FlowForm FORM, bool LINES>
__device__ __forceinline__ void flow_diagonal_task(const FlowArgs<T, LINES>& a, const int j, T* __restrict__ lds, int* shared) {
  using X = Mfma<T>;
  using acc_t = typename X::acc_t;
  using Sh = FlowShape<T, FORM>;
  constexpr bool SCALED = FORM == FLOW_SPD, PIVOT = FORM == FLOW_PIVOT;
  constexpr int BK = X::BK, KS = BK / 4;
  __builtin_amdgcn_s_setprio(3);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, g = lane >> 4;
  const int64_t j0 = (int64_t)j * LEAF;
  const int wl = a.w - j0 < LEAF ? (int)(a.w - j0) : LEAF;       // the leaf's order
  const FlowUnits units(wave, 1);
  acc_t x[NSUB], s[3];
  // entries of the leaf on and below its diagonal
  T* const leaf = a.P + j0 * (a.ld + 1);
#pragma unroll
  for (int u = 0; u < 3; ++u)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int grow = units.row[u] * SUB + X::acc_row(lane, r), gcol = units.col[u] * SUB + l16;
      s[u][r] = (u < units.count && grow < wl && gcol <= grow)
                    ? -__hip_atomic_load(leaf + (int64_t)grow * a.ld + gcol, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                    : T(0);
    }
  T v[NSUB][4];                      // the solved rows
  T* const solved = lds + Sh::SOLVED;
  T* const out = lds + Sh::DIAG_OUT + (wave & 3) * Sh::OUT;
  // to memory (wavefront 0's by wavefront 4)
  auto store_solved = [&] {
    if (j == 0 || wave < 1 || wave > 4) return;
    if (wave == 4) {
#pragma unroll
      for (int b = 0; b < NSUB; ++b) flow_solved_fetch(solved, 0, b, lane, v[b]);
    }
    flow_store_rows(a, a.P, j0 + (wave & 3) * SUB, j - 1, v, out, lane);
  };
  if (j > 0) {
#pragma unroll
    for (int b = 0; b < NSUB; ++b) x[b] = acc_t{0, 0, 0, 0};
    if (wave < 4) flow_load_rows(a, (const T*)a.P, j0 + wave * SUB, j - 1, x, lane);
    FlowOperands<T> of;
    of.row[0] = of.row[1] = a.P + j0 * a.ld;
    of.left[0] = of.left[1] = (int)(a.m - j0);
    of.col[0] = of.col[1] = a.P + (j0 - LEAF) * a.ld;
    of.counter[0] = j;
    of.counter[1] = j - 1;
    of.counter[2] = of.counter[3] = -1;
    if (!flow_accumulate<T, FORM, 1>(a, of, j - 1, true, x, s, lds, shared)) return;
    if (flow_wait_all(a, j - 1, -1, -1, -1, j, shared) < 0) return;
    const LeafOperands<T> ops{lds};
    FlowGather order;
    if (PIVOT && wave < 4) order.load((const int*)(a.perm + j0 - LEAF), lane);
    // (the wavefronts that have columns to reorder leave the inverses to the others)
    flow_stage_leaf(ops, (const T*)(a.P + (j0 - LEAF) * (a.ld + 1)), a.ld, PIVOT ? wave ^ 4 : wave, lane);
    T rinv[NSUB][4];
    if (wave < 4) load_row((const T*)(a.dinv + j0 - LEAF), g, LEAF, rinv);
    T d[NSUB][4];                    // the pivots in the order of the product below
    if constexpr (!SCALED) {
#pragma unroll
      for (int q = 0; q < NSUB; ++q)
        load4((const T*)(a.dvec + j0 - LEAF + q / (KS / 4) * BK + g * KS + q % (KS / 4) * 4), d[q]);
    }
    if (PIVOT && wave < 4) order.apply(a.pivot0 + j0 - LEAF, x, out, lane);
    __syncthreads();
    if (wave < 4) {
      flow_solve(ops, x, lane);
      // the solved rows go from the wavefronts that hold them to all through LDS
      flow_solved_put(solved, wave, x, rinv, v, lane);
    }
    __syncthreads();
    // off the chain: the solved tile to memory; with pivoting, where all wavefronts meet before the elimination
    // begins, beside that, and the multipliers' places cleared here
    if constexpr (PIVOT) {
      if (wave >= 1 && wave <= 4)
        for (int e = LEAF_TILE + tid - 64; e < 2 * LEAF_TILE; e += 256) lds[e] = T(0);
    } else {
      store_solved();
    }
    // its product with itself, the columns in the order of a slab
#pragma unroll
    for (int p = 0; p < LEAF / BK; ++p) {
#pragma unroll
      for (int u = 0; u < 3; ++u)
        if (u < units.count) {
          T fr[KS], fc[KS];
          flow_solved_slab<T, KS>(solved, units.row[u], p, l16, g, fr);
          flow_solved_slab<T, KS>(solved, units.col[u], p, l16, g, fc);
#pragma unroll
          for (int e = 0; e < KS; ++e)
            s[u] = X::mfma(SCALED ? fr[e] : fr[e] * d[p * (KS / 4) + e / 4][e % 4], fc[e], s[u]);
        }
    }
  }
  if constexpr (PIVOT) {
    // (the whole leaf is there behind the first barrier of leaf_factor_pivoted_body, and tile (j, j - 1) in
    // memory behind its second one)
#pragma unroll
    for (int u = 0; u < 3; ++u)
      if (u < units.count) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int row = units.row[u] * SUB + X::acc_row(lane, r), col = units.col[u] * SUB + l16;
          const T v = row < wl ? -s[u][r] : T(row == col ? 1 : 0);
          lds[row * LEAF_PAD + (col <= row ? col : LEAF)] = v;   // (or to the padding: no jump)
          lds[col * LEAF_PAD + (col <= row ? row : LEAF)] = v;
        }
      }
    leaf_factor_pivoted_body<T, true, true>(leaf, a.ld, wl, a.dvec + j0, a.dinv + j0, nullptr, a.perm + j0, a.pivot0 + j0,
                                            a.flags, lds, &a.sync->done[j], (unsigned)j, store_solved, j > 0);
  } else {
    // wavefront 0 goes on with its sub-block at once; the others' are there, and tile (j, j - 1) is
    // in memory, when it is through with that (the first barrier of leaf_factor_body)
#pragma unroll
    for (int u = 0; u < 3; ++u)
      if (u < units.count) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
          leaf_tile_put<T>(lds, units.row[u] * SUB + X::acc_row(lane, r), units.col[u] * SUB + l16, wl, -s[u][r]);
      }
    if (wave != 0) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    leaf_factor_body<T, true, true>(leaf, a.ld, wl, a.dvec + j0, a.dinv + j0, nullptr, a.pivot0 + j0, a.flags, lds,
                                    SCALED ? 1 : 0, &a.sync->done[j], (unsigned)j);
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (tid == 0) flow_publish(a, j, j + 1);
}

// General matrices: P M = L D U of the leaf, and the tiles left of it in both arrays, L's by
// wavefronts 0 to 3, U^T's by the others.
template <typename T, bool LINES>
__device__ __forceinline__ void flow_diagonal_general(const FlowArgs<T, LINES>& a, const int j, T* __restrict__ lds, int* shared) {
  using X = Mfma<T>;
  using acc_t = typename X::acc_t;
  using Sh = FlowShape<T, FLOW_GENERAL>;
  constexpr int BK = X::BK, KS = BK / 4;
  __builtin_amdgcn_s_setprio(3);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, g = lane >> 4;
  const int64_t j0 = (int64_t)j * LEAF;
  const int wl = a.w - j0 < LEAF ? (int)(a.w - j0) : LEAF;       // the leaf's order
  T* const Q = a.P + a.qoff;
  acc_t x[NSUB], s[3];
  T* const leaf = a.P + j0 * (a.ld + 1);
  const FlowUnits units(wave, 2);
  const int low = wave < 4 ? 0 : 1;                    // entries on the diagonal are the first array's
  {
    const T* D = leaf + (wave < 4 ? 0 : a.qoff);
#pragma unroll
    for (int u = 0; u < 3; ++u)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = units.row[u] * SUB + X::acc_row(lane, r), col = units.col[u] * SUB + l16;
        s[u][r] = u < units.count && row < wl && col + low <= row
                      ? -__hip_atomic_load(D + (int64_t)row * a.ld + col, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                      : T(0);
      }
  }
  if (j > 0) {
    T* const solved = lds + Sh::SOLVED;
    T* const rows = wave < 4 ? a.P : Q;
    const int64_t r16 = j0 + (wave & 3) * SUB;
    flow_load_rows(a, (const T*)rows, r16, j - 1, x, lane);
    FlowOperands<T> of;
    of.row[0] = a.P + j0 * a.ld;
    of.row[1] = Q + j0 * a.ld;
    of.left[0] = of.left[1] = (int)(a.m - j0);
    of.col[0] = Q + (j0 - LEAF) * a.ld;
    of.col[1] = a.P + (j0 - LEAF) * a.ld;
    of.counter[0] = j;
    of.counter[1] = a.order.ntr + j;
    of.counter[2] = j - 1;
    of.counter[3] = a.order.ntr + j - 1;
    if (!flow_accumulate<T, FLOW_GENERAL, 2>(a, of, j - 1, true, x, s, lds, shared)) return;
    if (flow_wait_all(a, j - 1, -1, -1, -1, j, shared) < 0) return;
    const LeafOperands<T> opsL{lds}, opsU{lds + LeafOperands<T>::ELEMS};
    const T* const before = a.P + (j0 - LEAF) * (a.ld + 1);
    FlowGather order;
    if (wave >= 4) order.load((const int*)(a.perm + j0 - LEAF), lane);
    flow_stage_both(opsL, opsU, before, before + a.qoff, a.ld, wave, lane);
    T rinv[NSUB][4], d[NSUB][4];
    load_row((const T*)(a.dinv + j0 - LEAF), g, LEAF, rinv);
#pragma unroll
    for (int q = 0; q < NSUB; ++q)
      load4((const T*)(a.dvec + j0 - LEAF + q / (KS / 4) * BK + g * KS + q % (KS / 4) * 4), d[q]);
    // (the places of the solved tiles are free)
    if (wave >= 4) order.apply(a.pivot0 + j0 - LEAF, x, solved + (wave & 3) * Sh::OUT, lane);
    __syncthreads();
    flow_solve(wave < 4 ? opsU : opsL, x, lane);
    T v[NSUB][4];
    flow_solved_put(solved, wave, x, rinv, v, lane);
    __syncthreads();
    // their product, the columns in the order of a slab
    const int mine0 = wave & 4, other0 = 4 - mine0;
#pragma unroll
    for (int p = 0; p < LEAF / BK; ++p) {
#pragma unroll
      for (int u = 0; u < 3; ++u)
        if (u < units.count) {
          T fr[KS], fc[KS];
          flow_solved_slab<T, KS>(solved, mine0 + units.row[u], p, l16, g, fr);
          flow_solved_slab<T, KS>(solved, other0 + units.col[u], p, l16, g, fc);
#pragma unroll
          for (int e = 0; e < KS; ++e) s[u] = X::mfma(fr[e] * d[p * (KS / 4) + e / 4][e % 4], fc[e], s[u]);
        }
    }
  }
#pragma unroll
  for (int u = 0; u < 3; ++u)
    if (u < units.count) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = units.row[u] * SUB + X::acc_row(lane, r), col = units.col[u] * SUB + l16;
        const int to_row = low ? col : row, to_col = low ? row : col;
        lds[to_row * LEAF_PAD + (col + low <= row ? to_col : LEAF)] = row < wl ? -s[u][r] : T(row == col ? 1 : 0);
      }
    }
  // The solved tiles go to memory beside the elimination, by the wavefront that is through with its columns of
  // it first: stored before, and waited for so that their counters can say so, they hold it up by 4 us.
  auto store_solved = [&] {
    if (j == 0) return;
    T* const solved = lds + Sh::SOLVED;
#pragma unroll 1
    for (int q = 0; q < 2 * NSUB; ++q) {
      T v[NSUB][4];
#pragma unroll
      for (int b = 0; b < NSUB; ++b) flow_solved_fetch(solved, q, b, lane, v[b]);
      flow_store_rows(a, q < NSUB ? a.P : Q, j0 + (q & (NSUB - 1)) * SUB, j - 1, v, lds + Sh::DIAG_OUT, lane);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if (lane == 0) {
      flow_publish(a, j, j);
      flow_publish(a, a.order.ntr + j, j);
    }
  };
  leaf_lu_body<T, FLOW_WAVES, true, true>(leaf, leaf + a.qoff, a.ld, wl, a.dvec + j0, a.dinv + j0, nullptr, nullptr,
                                          a.perm + j0, a.pivot0 + j0, a.flags, lds, store_solved);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (tid == 0) {
    flow_publish(a, a.order.ntr + j, j + 1);
    flow_publish(a, j, j + 1);
  }
}

// Starts on a page: its 47 to 64 KB of instructions nearly fill the instruction cache, and where in a page
// the code before it made it start moved the pivoted form in fp64 by 1.4 % (n = 6000, the same
// instructions 0x600 and 0xb00 behind a page's start 2391 and 2426 us, at its start 2392).
template <typename T, FlowForm FORM, bool LINES>
__attribute__((aligned(4096))) __global__ __launch_bounds__(FLOW_THREADS) void panel_flow_kernel(FlowArgs<T, LINES> a) {
  __shared__ __attribute__((aligned(16))) T lds[FlowShape<T, FORM>::LDS_ELEMS];
  __shared__ int shared[2];
  if (threadIdx.x == 0)
    shared[1] = (int)__hip_atomic_fetch_add(&a.sync->ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __syncthreads();
  int pair, array, j;
  const int kind = __builtin_amdgcn_readfirstlane(
      (int)a.order.task(__builtin_amdgcn_readfirstlane(shared[1]), pair, array, j));
  pair = __builtin_amdgcn_readfirstlane(pair);
  array = __builtin_amdgcn_readfirstlane(array);
  j = __builtin_amdgcn_readfirstlane(j);
  if (kind == FLOW_DIAGONAL) {
    if constexpr (FORM == FLOW_GENERAL) flow_diagonal_general<T>(a, j, lds, shared);
    else flow_diagonal_task<T, FORM>(a, j, lds, shared);
  } else if (kind == FLOW_ROWS2) {
    __builtin_amdgcn_s_setprio(2);
    flow_row2_task<T, FORM>(a, pair, array, j, lds, shared);
  } else if (kind == FLOW_ROWS) {
    __builtin_amdgcn_s_setprio(2);
    flow_row_task<T, FORM>(a, pair, array, j, lds, shared);
  }
}

// The words of FlowSync, n of them, to zero.
__global__ void flow_reset_kernel(unsigned* words, int n) {
  for (int q = blockIdx.x * blockDim.x + threadIdx.x; q < n; q += gridDim.x * blockDim.x) words[q] = 0u;
}

}  // namespace mdet
