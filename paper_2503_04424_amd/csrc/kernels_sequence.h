// Principal-minor sequence and the FLODANCE regression (Sec. 3.2, Alg. 2).
//
// The LDL^T factorisation yields the log-determinants of all leading principal
// blocks at once, ell_k = sum_{i<=k} log|D_ii| (Sec. 2.1: the diagonal factors give
// every leading principal minor), and Alg. 2 fits a curve to that sequence:
//
//   L_j = ell_{j d} / j,   n_j = n_0 + j   (j = 1 .. n_s - n_0)
//   y_j = n_j (n_j-1)^-1/2 (L_{n_j} - L_{n_0})
//   X_j1 = (n_j-1)^1/2,   X_j,i+1 = -(n_j-1)^-1/2 n_j^(1-i) logGamma(n_j+1),  i = 1 .. q+1
//   beta = argmin |X beta - y|_2,   (c_0, nu_0 .. nu_q) = beta
//   Lhat_n = L_{n_0} + c_0 (1 - 1/n) - sum_{i=1}^{q+1} nu_{i-1} n^-i logGamma(n+1)
//
// Kernels here: the running sum (a scan in two passes, three for long sequences), the
// least-squares problem as a tree of Householder QR factorisations of [X y] (one row per
// thread, 256 rows per workgroup; the normal equations X^T X of Alg. 2 would square a condition number
// that grows like n^q), and the evaluation of Lhat_n.  All arithmetic is fp64.
//
// The order of every sum is part of what the library returns: the coefficients of a fit answer
// to the last bits of R (two trees that are equally accurate in the column-scaled coordinates
// give vectors up to 1e-9 of their norm apart), so sums are formed in one order whatever the
// sizes: 16 entries, 256 of those, chunk after chunk in the scan; 64 lanes by halves, four
// wavefronts, 256 rows a workgroup in the fit.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mdet {

// ---------------------------------------------------------------------------
// ell_k = sum_{i<=k} log|d_i|
// ---------------------------------------------------------------------------
// A chunk of 4096 entries per workgroup: SEQ_THREADS threads take the logarithms, four entries
// each, and the first SEQ_SUMS of them add up SEQ_PER entries each, handed over through LDS
// (n = 500 000: 22.2 us with 16 logarithms in a row in each of 256 threads and always three
// passes, 13 now).
constexpr int SEQ_THREADS = 1024;
constexpr int SEQ_SUMS = 256;
constexpr int SEQ_PER = 16;
constexpr int SEQ_PAD = SEQ_PER + 1;
constexpr int SEQ_CHUNK = SEQ_SUMS * SEQ_PER;
// Up to so many chunks (n = 2 097 152) every workgroup of the last pass adds up the sums of the
// chunks before its own itself, beside its logarithms: two launches.  Beyond, a pass of its own
// does it once for all, since the work in every workgroup grows with their square.
constexpr int SEQ_DIRECT_CHUNKS = 512;

template <typename T>
__device__ __forceinline__ double log_abs_entry(const T* __restrict__ d, int64_t i, int64_t n) {
  return i < n ? log(fabs((double)d[i])) : 0.0;
}

// The logarithms of this workgroup's chunk into `tile`, then the running sums of SEQ_PER entries
// in place, by the first SEQ_SUMS threads; returns the thread's sum (the others': 0).  The
// caller's barrier publishes the running sums.
template <typename T>
__device__ __forceinline__ double seq_chunk_rows(const T* __restrict__ d, int64_t n, double* tile) {
  const int tid = threadIdx.x;
  const int64_t base = (int64_t)blockIdx.x * SEQ_CHUNK;
  constexpr int E = SEQ_CHUNK / SEQ_THREADS;
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int i = e * SEQ_THREADS + tid;
    tile[i / SEQ_PER * SEQ_PAD + i % SEQ_PER] = log_abs_entry(d, base + i, n);
  }
  __syncthreads();
  double s = 0.0;
  if (tid < SEQ_SUMS) {
    double* row = tile + tid * SEQ_PAD;
#pragma unroll
    for (int e = 0; e < SEQ_PER; ++e) {
      s += row[e];
      row[e] = s;
    }
  }
  return s;
}

// pass 1: one sum per chunk
template <typename T>
__global__ __launch_bounds__(SEQ_THREADS) void seq_chunk_sums_kernel(const T* __restrict__ d, int64_t n,
                                                                    double* __restrict__ sums) {
  __shared__ double tile[SEQ_SUMS * SEQ_PAD];
  __shared__ double red[SEQ_SUMS / 64];
  double s = seq_chunk_rows(d, n, tile);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (wave < SEQ_SUMS / 64) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off, 64);
    if (lane == 0) red[wave] = s;
  }
  __syncthreads();
  if (threadIdx.x == 0) sums[blockIdx.x] = ((red[0] + red[1]) + red[2]) + red[3];
}

// pass 2 (more than SEQ_DIRECT_CHUNKS chunks): exclusive running sum of the chunk sums, in
// order: one workgroup stages them through LDS, one thread adds them up, n / 4096 of them, so
// that its time grows with n (513 chunks and more)
constexpr int SEQ_OFFSET_THREADS = 256;
__global__ __launch_bounds__(SEQ_OFFSET_THREADS) void seq_chunk_offsets_kernel(double* __restrict__ sums,
                                                                              int64_t nchunks) {
  constexpr int M = 4 * SEQ_OFFSET_THREADS;
  __shared__ double tile[M];
  __shared__ double carry;
  if (threadIdx.x == 0) carry = 0.0;
  for (int64_t base = 0; base < nchunks; base += M) {
    const int64_t m = nchunks - base < M ? nchunks - base : M;
    for (int i = threadIdx.x; i < m; i += SEQ_OFFSET_THREADS) tile[i] = sums[base + i];
    __syncthreads();
    if (threadIdx.x == 0) {
      double run = carry;
      for (int i = 0; i < m; ++i) {
        const double v = tile[i];
        tile[i] = run;
        run += v;
      }
      carry = run;
    }
    __syncthreads();
    for (int i = threadIdx.x; i < m; i += SEQ_OFFSET_THREADS) sums[base + i] = tile[i];
    __syncthreads();
  }
}

// last pass: running sum inside each chunk on top of its offset; `offsets` holds the chunk sums
// themselves (DIRECT: added up here in the same order, by a wavefront that has no rows to sum)
// or the offsets
template <typename T, bool DIRECT>
__global__ __launch_bounds__(SEQ_THREADS) void seq_running_sum_kernel(const T* __restrict__ d, int64_t n,
                                                                     const double* __restrict__ offsets,
                                                                     double* __restrict__ ell) {
  __shared__ double tile[SEQ_SUMS * SEQ_PAD];
  __shared__ double tsum[2][SEQ_SUMS];
  __shared__ double before[DIRECT ? SEQ_DIRECT_CHUNKS : 1];
  __shared__ double offset;
  const int tid = threadIdx.x, nb = blockIdx.x;
  if constexpr (DIRECT) {
    if (tid < nb) before[tid] = offsets[tid];          // nb < SEQ_DIRECT_CHUNKS <= SEQ_THREADS
  }
  const double s = seq_chunk_rows(d, n, tile);          // (a barrier inside)
  if (tid < SEQ_SUMS) tsum[0][tid] = s;
  if (tid == SEQ_THREADS - 64) {
    double run = 0.0;
    if constexpr (DIRECT) {
#pragma unroll 8
      for (int c = 0; c < nb; ++c) run += before[c];
    } else {
      run = offsets[nb];
    }
    offset = run;
  }
  __syncthreads();
  // Hillis-Steele scan of the SEQ_SUMS thread sums
  int cur = 0;
#pragma unroll
  for (int off = 1; off < SEQ_SUMS; off <<= 1) {
    if (tid < SEQ_SUMS) {
      const double add = tid >= off ? tsum[cur][tid - off] : 0.0;
      tsum[cur ^ 1][tid] = tsum[cur][tid] + add;
    }
    cur ^= 1;
    __syncthreads();
  }
  const int64_t base = (int64_t)nb * SEQ_CHUNK;
  constexpr int E = SEQ_CHUNK / SEQ_THREADS;
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int i = e * SEQ_THREADS + tid, row = i / SEQ_PER;
    const double start = offset + (row > 0 ? tsum[cur][row - 1] : 0.0);
    if (base + i < n) ell[base + i] = start + tile[row * SEQ_PAD + i % SEQ_PER];
  }
}

// ---------------------------------------------------------------------------
// least squares by a tree of Householder QR factorisations
// ---------------------------------------------------------------------------
constexpr int FLO_MAX_Q = 10;
constexpr int FLO_MAX_COLS = FLO_MAX_Q + 3;      // q + 2 covariates and y
constexpr int FLO_ROWS = 256;                    // rows per workgroup = threads

// What the fit leaves in device memory: beta[0 .. q+1] = (c_0, nu_0 .. nu_q), then
// L_{n_0}, then the residual norm |X beta - y|_2.
struct FloProblem {
  const double* ell;
  int64_t d, n0, ns;
  int q;
};

// Row r (0-based) of [X y] of Alg. 2, P = q + 2 covariates then y.
__device__ __forceinline__ void flo_make_row(const FloProblem& pb, int64_t r, int ncols, double* row) {
  const double Ln0 = pb.ell[pb.n0 * pb.d - 1] / (double)pb.n0;
  const int64_t nj_i = pb.n0 + 1 + r;
  const double nj = (double)nj_i;
  const double Lnj = pb.ell[nj_i * pb.d - 1] / nj;
  const double root = sqrt(nj - 1.0);
  const double lg = lgamma(nj + 1.0);
  row[0] = root;
  double pw = 1.0;                                // n_j^(i-1)
  for (int i = 1; i < ncols - 1; ++i) {
    row[i] = -lg / (root * pw);
    pw *= nj;
  }
  row[ncols - 1] = nj / root * (Lnj - Ln0);
}

// Sums over the 64 lanes of four values at once: row 0 of 16 lanes ends up with that of p0, rows
// 1, 2 and 3 with those of p2, p1 and p3.  Lanes 32 apart are added first, then 16, 8, 4, 2 and 1:
// the order of an exchange by halves, with two values sharing a register after the first step
// and four after the second (one sum through LDS shuffles costs as much as eight of these).
// Addition commutes, so a step leaves the same value in all lanes that it has combined; that is
// why a rotation serves for the exchange of lanes 8 and 4 apart.
__device__ __forceinline__ void flo_swap32(double& a, double& b) {
  const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)__double2loint(a), (unsigned)__double2loint(b), false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)__double2hiint(a), (unsigned)__double2hiint(b), false, false);
  a = __hiloint2double((int)hi[0], (int)lo[0]);
  b = __hiloint2double((int)hi[1], (int)lo[1]);
}
__device__ __forceinline__ void flo_swap16(double& a, double& b) {
  const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)__double2loint(a), (unsigned)__double2loint(b), false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)__double2hiint(a), (unsigned)__double2hiint(b), false, false);
  a = __hiloint2double((int)hi[0], (int)lo[0]);
  b = __hiloint2double((int)hi[1], (int)lo[1]);
}
__device__ __forceinline__ double flo_wave_sum4(double p0, double p1, double p2, double p3) {
  flo_swap32(p0, p1);      // [p0 lower half, p1 lower half], [p0 upper half, p1 upper half]
  flo_swap32(p2, p3);
  double u = p0 + p1, v = p2 + p3;
  flo_swap16(u, v);        // the even rows of both, the odd rows of both
  u += v;
#define MDET_FLO_ADD(CTRL) \
  u += __longlong_as_double(__builtin_amdgcn_update_dpp(0ll, __double_as_longlong(u), CTRL, 0xF, 0xF, true))
  MDET_FLO_ADD(0x128);    // rotation by 8 inside each row of 16 lanes
  MDET_FLO_ADD(0x124);    // by 4 (the row repeats itself after 8)
  MDET_FLO_ADD(0x4E);     // lanes 2 3 0 1 of each four
  MDET_FLO_ADD(0xB1);     // lanes 1 0 3 2
#undef MDET_FLO_ADD
  return u;
}

// One workgroup reduces up to FLO_ROWS rows of NC columns to the upper-triangular
// NC x NC factor R of their QR factorisation (Householder reflections; the
// orthogonal factor is never formed).  Level 0 builds its rows from ell, higher
// levels read them from `in` (row-major, nrows x NC: the stacked R factors of the
// level below).  out: NC x NC per workgroup, row-major, zeros below the
// diagonal.  If `coef` is given (last level, one workgroup), thread 0 also solves
// R[0:P, 0:P] beta = R[0:P, P] and writes beta, L_{n_0} and |R[P][P]|.
// The number of columns is a template parameter, so that only columns there are take part; a
// reflection is one block reduction of all column dot products at once and bounds the kernel.
// Which product is fused with which sum is written out: the result must not depend on how the
// compiler contracts this form of the loops (see the top of the file).
// Measured, q = 4, three levels for 50 000 samples: 70 us with 13 columns always and one sum
// at a time through shuffles, 18.6 now (q = 10: 134 -> 41).  Four rows a thread and two levels
// took 17.1, but in another order of summation.
template <int NC>
__global__ __launch_bounds__(FLO_ROWS) void flo_qr_kernel(FloProblem pb, const double* __restrict__ in,
                                                         int64_t nrows, double* __restrict__ out,
                                                         double* __restrict__ coef) {
  __shared__ double red[2][NC][4];
  __shared__ double pivot_row[2][NC];
  __shared__ double Rs[NC][NC];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int column_of_row = ((lane >> 5) & 1) + 2 * ((lane >> 4) & 1);     // see flo_wave_sum4
  const int64_t r = (int64_t)blockIdx.x * FLO_ROWS + tid;
  double a[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) a[c] = 0.0;
  if (r < nrows) {
    if (in == nullptr) {
      flo_make_row(pb, r, NC, a);
    } else {
#pragma unroll
      for (int c = 0; c < NC; ++c) a[c] = in[r * NC + c];
    }
  }
#pragma unroll
  for (int k = 0; k < NC; ++k) {
    const int buf = k & 1;
    // dot products of column k with columns k.. over rows k.. (row t = thread t)
    const bool in_play = tid >= k;
    const double x = a[k];
#pragma unroll
    for (int c = k; c < NC; c += 4) {
      double p[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) p[e] = c + e < NC && in_play ? x * a[c + e < NC ? c + e : k] : 0.0;
      const double sum = flo_wave_sum4(p[0], p[1], p[2], p[3]);
      const int mine = c + column_of_row;
      if ((lane & 15) == 0 && mine < NC) red[buf][mine][wave] = sum;
    }
    if (tid == k) {
#pragma unroll
      for (int c = k; c < NC; ++c) pivot_row[buf][c] = a[c];
    }
    __syncthreads();
    const double sigma = ((red[buf][k][0] + red[buf][k][1]) + red[buf][k][2]) + red[buf][k][3];
    const double xk = pivot_row[buf][k];
    // reflector v = x - alpha e_k, alpha = -sign(x_k) |x|; H = I - 2 v v^T / (v^T v)
    const double alpha = xk > 0.0 ? -sqrt(sigma) : sqrt(sigma);
    const double vtv = 2.0 * fma(-alpha, xk, sigma);
    if (vtv > 0.0) {
      const double v = in_play ? (tid == k ? x - alpha : x) : 0.0;
#pragma unroll
      for (int c = k + 1; c < NC; ++c) {
        const double xc = ((red[buf][c][0] + red[buf][c][1]) + red[buf][c][2]) + red[buf][c][3];
        const double vta = fma(-alpha, pivot_row[buf][c], xc);      // v^T A_c
        a[c] = fma(-(2.0 * vta / vtv), v, a[c]);
      }
    }
    // column k becomes (.., alpha, 0, ..)
    if (in_play) a[k] = tid == k ? (vtv > 0.0 ? alpha : xk) : 0.0;
  }
  // rows 0 .. NC-1 now hold R
  if (tid < NC) {
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const double v = c >= tid ? a[c] : 0.0;
      out[((int64_t)blockIdx.x * NC + tid) * NC + c] = v;
      Rs[tid][c] = v;
    }
  }
  if (coef != nullptr) {
    __syncthreads();
    if (tid == 0) {
      constexpr int P = NC - 1;
      double beta[P];
#pragma unroll
      for (int i = P - 1; i >= 0; --i) {
        double s = Rs[i][P];
#pragma unroll
        for (int c = i + 1; c < P; ++c) s = fma(-Rs[i][c], beta[c], s);
        beta[i] = s / Rs[i][i];
        coef[i] = beta[i];
      }
      coef[P] = pb.ell[pb.n0 * pb.d - 1] / (double)pb.n0;
      coef[P + 1] = fabs(Rs[P][P]);
    }
  }
}

// Lhat_n for each n in n_values (last step of Alg. 2)
__global__ void flo_eval_kernel(const double* __restrict__ coef, int q, const double* __restrict__ n_values,
                                int64_t count, double* __restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= count) return;
  const double n = n_values[i];
  const double lg = lgamma(n + 1.0);
  double acc = coef[q + 2] + coef[0] * (1.0 - 1.0 / n);
  double pw = n;                                   // n^i
  for (int t = 1; t <= q + 1; ++t) {
    acc -= coef[t] * lg / pw;
    pw *= n;
  }
  out[i] = acc;
}

}  // namespace mdet
