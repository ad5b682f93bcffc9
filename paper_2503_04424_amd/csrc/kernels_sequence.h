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
// least-squares problem as a tree of Householder QR factorisations of [X y] (four rows per
// thread, 1024 rows per workgroup; the normal equations X^T X of Alg. 2 would square a condition number
// that grows like n^q), and the evaluation of Lhat_n.  All arithmetic is fp64.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mdet {

// ---------------------------------------------------------------------------
// ell_k = sum_{i<=k} log|d_i|
// ---------------------------------------------------------------------------
constexpr int SEQ_THREADS = 256;
// Entries per thread.  Up to SEQ_FINE_CHUNKS chunks of four entries a thread, every workgroup of
// the last pass adds the sums of the chunks before its own itself: two launches, and four
// times as many workgroups for the logarithms (n = 500 000: 23.4 -> 11.8 us of kernels).
// Beyond, 16 entries a thread and a pass for the offsets, since adding up all chunks in every
// workgroup grows with their square.
constexpr int SEQ_PER_FINE = 4, SEQ_PER_COARSE = 16;
constexpr int SEQ_FINE_CHUNKS = 2048;

// Sum of `v` over the workgroup's 256 threads, the same value in every thread; the
// four wavefronts' sums are added in a fixed order.  `red`: 4 doubles of LDS; two
// barriers inside.
__device__ __forceinline__ double block_sum256(double v, double* red) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) red[wave] = v;
  __syncthreads();
  return ((red[0] + red[1]) + red[2]) + red[3];
}

template <typename T>
__device__ __forceinline__ double log_abs_entry(const T* __restrict__ d, int64_t i, int64_t n) {
  return i < n ? log(fabs((double)d[i])) : 0.0;
}

// pass 1: one sum per chunk
template <typename T, int PER>
__global__ __launch_bounds__(SEQ_THREADS) void seq_chunk_sums_kernel(const T* __restrict__ d, int64_t n,
                                                                    double* __restrict__ sums) {
  __shared__ double red[4];
  const int64_t base = ((int64_t)blockIdx.x * SEQ_THREADS + threadIdx.x) * PER;
  double s = 0.0;
#pragma unroll
  for (int e = 0; e < PER; ++e) s += log_abs_entry(d, base + e, n);
  s = block_sum256(s, red);
  if (threadIdx.x == 0) sums[blockIdx.x] = s;
}

// pass 2 (coarse chunks only): exclusive running sum of the chunk sums, in order (a few hundred at most):
// one workgroup stages them through LDS, one thread adds them up
__global__ __launch_bounds__(SEQ_THREADS) void seq_chunk_offsets_kernel(double* __restrict__ sums,
                                                                       int64_t nchunks) {
  __shared__ double tile[4 * SEQ_THREADS];
  __shared__ double carry;
  if (threadIdx.x == 0) carry = 0.0;
  for (int64_t base = 0; base < nchunks; base += 4 * SEQ_THREADS) {
    const int64_t m = nchunks - base < 4 * SEQ_THREADS ? nchunks - base : 4 * SEQ_THREADS;
    for (int i = threadIdx.x; i < m; i += SEQ_THREADS) tile[i] = sums[base + i];
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
    for (int i = threadIdx.x; i < m; i += SEQ_THREADS) sums[base + i] = tile[i];
    __syncthreads();
  }
}

// last pass: running sum inside each chunk on top of its offset; `offsets` holds the offsets
// (coarse chunks) or the chunk sums themselves, which are added up here (fine chunks)
template <typename T, int PER>
__global__ __launch_bounds__(SEQ_THREADS) void seq_running_sum_kernel(const T* __restrict__ d, int64_t n,
                                                                     const double* __restrict__ offsets,
                                                                     double* __restrict__ ell) {
  __shared__ double tsum[SEQ_THREADS];
  __shared__ double red[4];
  const int tid = threadIdx.x;
  const int64_t base = ((int64_t)blockIdx.x * SEQ_THREADS + tid) * PER;
  double offset;
  if constexpr (PER == SEQ_PER_FINE) {
    double mine = 0.0;
    for (int64_t c = tid; c < blockIdx.x; c += SEQ_THREADS) mine += offsets[c];
    offset = block_sum256(mine, red);
  } else {
    offset = offsets[blockIdx.x];
  }
  double v[PER];
  double s = 0.0;
#pragma unroll
  for (int e = 0; e < PER; ++e) {
    s += log_abs_entry(d, base + e, n);
    v[e] = s;
  }
  tsum[tid] = s;
  __syncthreads();
  // Hillis-Steele scan of the 256 thread sums
  for (int off = 1; off < SEQ_THREADS; off <<= 1) {
    const double add = tid >= off ? tsum[tid - off] : 0.0;
    __syncthreads();
    tsum[tid] += add;
    __syncthreads();
  }
  const double before = offset + (tid > 0 ? tsum[tid - 1] : 0.0);
#pragma unroll
  for (int e = 0; e < PER; ++e)
    if (base + e < n) ell[base + e] = before + v[e];
}

// ---------------------------------------------------------------------------
// least squares by a tree of Householder QR factorisations
// ---------------------------------------------------------------------------
constexpr int FLO_MAX_Q = 10;
constexpr int FLO_MAX_COLS = FLO_MAX_Q + 3;      // q + 2 covariates and y
constexpr int FLO_THREADS = 256;
constexpr int FLO_PER = 4;                       // rows per thread
constexpr int FLO_ROWS = FLO_THREADS * FLO_PER;  // rows per workgroup

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

// Sum over the 64 lanes, in lane 63: inside each row of 16 lanes, then the last lane of a row
// handed on (the exchange pattern of a maximum over the wavefront; a shuffle through LDS
// costs four times as much).
__device__ __forceinline__ double flo_wave_sum(double v) {
#define MDET_FLO_ADD(CTRL, ROWS)                                                                            \
  v += __longlong_as_double(__builtin_amdgcn_update_dpp(0ll, __double_as_longlong(v), CTRL, ROWS, 0xF, true))
  MDET_FLO_ADD(0xB1, 0xF);     // lanes 1 0 3 2 of each four
  MDET_FLO_ADD(0x4E, 0xF);     // lanes 2 3 0 1
  MDET_FLO_ADD(0x141, 0xF);    // mirror inside each eight
  MDET_FLO_ADD(0x140, 0xF);    // mirror inside each sixteen
  MDET_FLO_ADD(0x142, 0xA);    // lane 15 -> rows 1 and 3 (the others receive 0)
  MDET_FLO_ADD(0x143, 0xC);    // lane 31 -> rows 2 and 3
#undef MDET_FLO_ADD
  return v;
}

// One workgroup reduces up to FLO_ROWS rows of NC columns to the upper-triangular
// NC x NC factor R of their QR factorisation (Householder reflections; the
// orthogonal factor is never formed).  Level 0 builds its rows from ell, higher
// levels read them from `in` (row-major, nrows x NC: the stacked R factors of the
// level below).  out: NC x NC per workgroup, row-major, zeros below the
// diagonal.  If `coef` is given (last level, one workgroup), thread 0 also solves
// R[0:P, 0:P] beta = R[0:P, P] and writes beta, L_{n_0} and |R[P][P]|.
// Thread t holds rows t, t + 256, ...; the number of columns is a template parameter, so that
// only columns there are take part.  A reflection is one block reduction of all column dot
// products at once and bounds the kernel: four rows a thread make the tree two levels high
// at 50 000 samples instead of three.  Measured there, q = 4: 3 x 23.9 us with one row a
// thread, the sums by shuffles and always 13 columns; 2 x 9.6 us now.
template <int NC>
__global__ __launch_bounds__(FLO_THREADS) void flo_qr_kernel(FloProblem pb, const double* __restrict__ in,
                                                            int64_t nrows, double* __restrict__ out,
                                                            double* __restrict__ coef) {
  __shared__ double red[2][NC][4];
  __shared__ double pivot_row[2][NC];
  __shared__ double Rs[NC][NC];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  double a[FLO_PER][NC];
#pragma unroll
  for (int s = 0; s < FLO_PER; ++s) {
    const int64_t r = (int64_t)blockIdx.x * FLO_ROWS + s * FLO_THREADS + tid;
#pragma unroll
    for (int c = 0; c < NC; ++c) a[s][c] = 0.0;
    if (r < nrows) {
      if (in == nullptr) {
        flo_make_row(pb, r, NC, a[s]);
      } else {
#pragma unroll
        for (int c = 0; c < NC; ++c) a[s][c] = in[r * NC + c];
      }
    }
  }
#pragma unroll
  for (int k = 0; k < NC; ++k) {
    const int buf = k & 1;
    // dot products of column k with columns k.. over rows k..; row k is thread k's first
    const bool in_play = tid >= k;
    double x[FLO_PER];
#pragma unroll
    for (int s = 0; s < FLO_PER; ++s) x[s] = s > 0 || in_play ? a[s][k] : 0.0;
#pragma unroll
    for (int c = k; c < NC; ++c) {
      double p = x[0] * a[0][c];
#pragma unroll
      for (int s = 1; s < FLO_PER; ++s) p = fma(x[s], a[s][c], p);
      p = flo_wave_sum(p);
      if (lane == 63) red[buf][c][wave] = p;
    }
    if (tid == k) {
#pragma unroll
      for (int c = k; c < NC; ++c) pivot_row[buf][c] = a[0][c];
    }
    __syncthreads();
    const double sigma = ((red[buf][k][0] + red[buf][k][1]) + red[buf][k][2]) + red[buf][k][3];
    const double xk = pivot_row[buf][k];
    // reflector v = x - alpha e_k, alpha = -sign(x_k) |x|; H = I - 2 v v^T / (v^T v)
    const double alpha = xk > 0.0 ? -sqrt(sigma) : sqrt(sigma);
    const double vtv = 2.0 * (sigma - alpha * xk);
    if (vtv > 0.0) {
      x[0] = tid == k ? x[0] - alpha : x[0];
      const double scale = 2.0 / vtv;
#pragma unroll
      for (int c = k + 1; c < NC; ++c) {
        const double xc = ((red[buf][c][0] + red[buf][c][1]) + red[buf][c][2]) + red[buf][c][3];
        const double vta = xc - alpha * pivot_row[buf][c];      // v^T A_c
        const double f = scale * vta;
#pragma unroll
        for (int s = 0; s < FLO_PER; ++s) a[s][c] -= f * x[s];
      }
    }
    // column k becomes (.., alpha, 0, ..)
    if (in_play) a[0][k] = tid == k ? (vtv > 0.0 ? alpha : xk) : 0.0;
#pragma unroll
    for (int s = 1; s < FLO_PER; ++s) a[s][k] = 0.0;
  }
  // rows 0 .. NC-1 now hold R
  if (tid < NC) {
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const double v = c >= tid ? a[0][c] : 0.0;
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
        for (int c = i + 1; c < P; ++c) s -= Rs[i][c] * beta[c];
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
