// Construction of the impulse responses h_k from a TVIR (section 4): the L2
// projection of every TVIR row onto the span of the windows (section 4.2,
// the B-spline case of Corollary 4.3) and the interpolation at m nodes
// (section 4.4).  For a lag row T(x, .):
//   projection:     (W W^T) c(x) = W T(x, .)^T
//   interpolation:  E c(x) = (T(x, y_i))_i,   E[i][k] = w_k(y_i)
// and h_k[x] = c_k(x) / n.
//
// The contraction W T^T (rows x n times n x m) is the one dense product of
// the path: it runs on the matrix cores in FP32 (v_mfma_f32_16x16x4f32), split
// along n into chunks whose partial sums are added in float64; the m x m
// inverse or factorisation and the per-row solves are float64.
#include "pc_internal.hpp"
#include "project_tile.hpp"

namespace pc {

typedef float floatx4 __attribute__((ext_vector_type(4)));

// part[seg][r][c] = sum over the segment's j of A[r][j] B[c][j], in float64
// from FP32 sums of at most GEMM_CHUNK terms.  A: the rows x K TVIR band
// followed by the cols x K windows themselves (their Gram matrix), B: the
// windows; row-major with K contiguous, K % 16 == 0, 16-byte aligned rows.
//
// Bound by streaming the band from HBM once.  A workgroup (4 waves) takes
// GEMM_ROWS rows and 32 columns and walks its segment in stages of GEMM_KT
// samples: every row's stage is 256 contiguous bytes (16 lanes of 16 bytes;
// loads of 64 bytes per row, straight into MFMA operands, reached 4.1 TB/s),
// held in registers two stages ahead, then in one of two LDS buffers, where
// 16-byte chunk c of row r sits at c ^ (r mod 16), so that the 16 rows of an
// MFMA operand hit different banks.  48 KB of LDS: three workgroups per CU.
// Lane (i, g) feeds 4 consecutive k of its row and columns to 4 MFMA steps,
// the same k on both operands.  Workgroups of one segment are numbered
// together, so that the windows' segment stays in every L2.  Measured (23595
// lags x 65536 positions, 32 windows): 1517 us and 93 us for the Gram matrix
// with 64-byte row loads, 1146 us (5.4 TB/s, the rate of a large copy) here
// for both.
constexpr int GEMM_CPR = GEMM_KT / 4;  // 16-byte chunks per row and stage
__global__ __launch_bounds__(256) void k_gemm_nt_f32(const float* __restrict__ A, int64_t rows,
                                                     const float* __restrict__ B, int cols, int64_t K,
                                                     int seg_stages, double* __restrict__ part) {
  constexpr int AQ = GEMM_ROWS * GEMM_CPR / 256, BQ = GEMM_COLS * GEMM_CPR / 256;  // chunks per thread
  static_assert(GEMM_CPR == 16 && GEMM_ROWS == 64 && GEMM_COLS == 32, "tile of the lane mapping below");
  __shared__ floatx4 As[2][GEMM_ROWS * GEMM_CPR], Bs[2][GEMM_COLS * GEMM_CPR];
  const int tid = (int)threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int c = tid & 15, r = tid >> 4;  // load mapping: chunk c of rows r + 16 j
  const int64_t band_tiles = (rows + GEMM_ROWS - 1) / GEMM_ROWS;
  const bool gram = (int64_t)blockIdx.x >= band_tiles;
  const int64_t t0 = (gram ? blockIdx.x - band_tiles : blockIdx.x) * GEMM_ROWS;  // first row of the tile
  const int64_t have = gram ? cols : rows;
  const int c0 = (int)blockIdx.y * GEMM_COLS;
  const int64_t k_begin = (int64_t)blockIdx.z * seg_stages * GEMM_KT;
  const int64_t k_left = K - k_begin;
  const int ns = gemm_stages(k_left, seg_stages);
  // rows and columns past the last read the last one; their sums are not stored
  const float* ap[AQ];
  const float* bp[BQ];
#pragma unroll
  for (int j = 0; j < AQ; ++j) {
    const int64_t row = t0 + r + 16 * j < have ? t0 + r + 16 * j : have - 1;
    ap[j] = (gram ? B : A) + row * K + k_begin;
  }
#pragma unroll
  for (int j = 0; j < BQ; ++j) {
    const int col = c0 + r + 16 * j < cols ? c0 + r + 16 * j : cols - 1;
    bp[j] = B + (int64_t)col * K + k_begin;
  }
  floatx4 ra0[AQ], rb0[BQ], ra1[AQ], rb1[BQ];
  auto load = [&](floatx4(&a)[AQ], floatx4(&b)[BQ], int s) {
    // (stages past the segment's last are loaded and not used)
    const int64_t o = gemm_chunk_offset(s, c, k_left);
#pragma unroll
    for (int j = 0; j < AQ; ++j) a[j] = *reinterpret_cast<const floatx4*>(ap[j] + o);
#pragma unroll
    for (int j = 0; j < BQ; ++j) b[j] = *reinterpret_cast<const floatx4*>(bp[j] + o);
  };
  auto put = [&](int buf, const floatx4(&a)[AQ], const floatx4(&b)[BQ], int s) {
    // chunks past the row's end count as zero on both sides: a NaN or an
    // infinity read in their place would turn the other side's zeros into NaN
    const bool in = gemm_chunk_inside(s, c, k_left);
    const floatx4 zero{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < AQ; ++j)
      As[buf][(r + 16 * j) * GEMM_CPR + (c ^ r)] = in ? a[j] : zero;  // (r + 16 j) mod 16 = r
#pragma unroll
    for (int j = 0; j < BQ; ++j) Bs[buf][(r + 16 * j) * GEMM_CPR + (c ^ r)] = in ? b[j] : zero;
  };
  const int g = lane >> 4, li = lane & 15;
  floatx4 acc0{0.f, 0.f, 0.f, 0.f}, acc1{0.f, 0.f, 0.f, 0.f};
  double sum0[4] = {0., 0., 0., 0.}, sum1[4] = {0., 0., 0., 0.};
  auto compute = [&](int buf) {
    const floatx4* as = As[buf] + (16 * wave + li) * GEMM_CPR;
    const floatx4* b0 = Bs[buf] + li * GEMM_CPR;
    const floatx4* b1 = b0 + 16 * GEMM_CPR;
#pragma unroll
    for (int q = 0; q < GEMM_CPR / 4; ++q) {
      const int pos = (4 * q + g) ^ li;
      const floatx4 a = as[pos], x = b0[pos], y = b1[pos];
      acc0 = __builtin_amdgcn_mfma_f32_16x16x4f32(a.x, x.x, acc0, 0, 0, 0);
      acc1 = __builtin_amdgcn_mfma_f32_16x16x4f32(a.x, y.x, acc1, 0, 0, 0);
      acc0 = __builtin_amdgcn_mfma_f32_16x16x4f32(a.y, x.y, acc0, 0, 0, 0);
      acc1 = __builtin_amdgcn_mfma_f32_16x16x4f32(a.y, y.y, acc1, 0, 0, 0);
      acc0 = __builtin_amdgcn_mfma_f32_16x16x4f32(a.z, x.z, acc0, 0, 0, 0);
      acc1 = __builtin_amdgcn_mfma_f32_16x16x4f32(a.z, y.z, acc1, 0, 0, 0);
      acc0 = __builtin_amdgcn_mfma_f32_16x16x4f32(a.w, x.w, acc0, 0, 0, 0);
      acc1 = __builtin_amdgcn_mfma_f32_16x16x4f32(a.w, y.w, acc1, 0, 0, 0);
    }
  };
  auto flush = [&]() {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      sum0[i] += (double)acc0[i];
      sum1[i] += (double)acc1[i];
      acc0[i] = acc1[i] = 0.f;
    }
  };
  // stage s: stage s + 1 goes from its registers to the other buffer, whose
  // readers passed the barrier before; stage s + 3 is loaded in their place
  auto stage = [&](int s, floatx4(&a)[AQ], floatx4(&b)[BQ], int buf) {
    put(buf ^ 1, a, b, s + 1);
    load(a, b, s + 3);
    compute(buf);
    if ((s + 1) % (GEMM_CHUNK / GEMM_KT) == 0) flush();
    __syncthreads();
  };
  load(ra0, rb0, 0);
  load(ra1, rb1, 1);
  put(0, ra0, rb0, 0);
  load(ra0, rb0, 2);
  __syncthreads();
  for (int s = 0; s < ns; s += 2) {
    stage(s, ra1, rb1, 0);
    if (s + 1 < ns) stage(s + 1, ra0, rb0, 1);
  }
  flush();
  // output block element (i, j) sits in lane j + 16 (i / 4), item i % 4
  double* P = part + ((int64_t)blockIdx.z * (rows + cols) + (gram ? rows : 0)) * cols;
  const int ca = c0 + li, cb = ca + 16;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int64_t row = t0 + 16 * wave + 4 * g + i;
    if (row < have) {
      if (ca < cols) P[row * cols + ca] = sum0[i];
      if (cb < cols) P[row * cols + cb] = sum1[i];
    }
  }
}

// Inverse of the Gram matrix (m x m, m <= CONSTRUCT_MAX_M; the last m rows of
// the contraction, summed over its segments) by Gauss-Jordan elimination in
// LDS, one workgroup: every step updates the whole matrix in parallel (the
// triangular factorisation and solves it replaces were chains of dependent
// LDS reads: 40 us at m = 32, 24 here; 38 with 256 threads).  Without exchanges, as the matrix
// is symmetric positive definite; step p's pivot is the one of its Cholesky
// factorisation.  *fail = 1 if a pivot is not above 1e-12 of its diagonal
// entry (the windows are numerically dependent).
__global__ __launch_bounds__(1024) void k_gram_inverse(const double* __restrict__ part, int segs, int64_t rows, int m,
                                                       double* __restrict__ inv, int* __restrict__ fail) {
  __shared__ double S[CONSTRUCT_MAX_M * CONSTRUCT_MAX_M];
  __shared__ double diag[CONSTRUCT_MAX_M];
  const int nt = (int)blockDim.x, rs = nt >> 5;
  const int ti = (int)threadIdx.x >> 5, tj = (int)threadIdx.x & 31;  // element (ti + rs a, tj + 32 b)
  for (int i = ti; i < m; i += rs)
    for (int j = tj; j < m; j += 32) {
      const double* g = part + (rows * m + (int64_t)i * m + j);
      double v = 0.0;
#pragma unroll 4
      for (int q = 0; q < segs; ++q) v += g[(int64_t)q * (rows + m) * m];
      S[i * m + j] = v;
      if (i == j) diag[i] = v;
    }
  int bad = 0;
  __syncthreads();
  for (int p = 0; p < m; ++p) {
    double d = S[p * m + p];
    if (!(d > 1e-12 * diag[p])) {
      bad = 1;
      d = 1.0;
    }
    const double rd = 1.0 / d;
    for (int i = ti; i < m; i += rs) {
      const double f = S[i * m + p] * rd;
      for (int j = tj; j < m; j += 32)
        if (i != p && j != p) S[i * m + j] -= f * S[p * m + j];
    }
    __syncthreads();
    for (int i = (int)threadIdx.x; i < m; i += nt) {
      if (i == p) {
        S[p * m + p] = rd;
      } else {
        S[i * m + p] *= -rd;
        S[p * m + i] *= rd;
      }
    }
    __syncthreads();
  }
  for (int i = (int)threadIdx.x; i < m * m; i += nt) inv[i] = S[i];
  if (threadIdx.x == 0) *fail = bad;
}

// h[k][lags[r]] = sum_j inv[k][j] b_r[j] / n, b_r the contraction's row r
// summed over its segments (float64): PROJECT_ROWS rows per workgroup, their
// right-hand sides in LDS, a wave per k with a row per lane (consecutive lags
// mostly, so the stores are contiguous; inv is read uniformly).  One thread
// per row with its vector in memory took 105 us (23595 rows, m = 32) after
// 33 us of summing; 15 us here, sums included.
constexpr int PROJECT_ROWS = 64;
__global__ __launch_bounds__(256) void k_project_solve(const double* __restrict__ part, int segs, int64_t rows, int m,
                                                       const double* __restrict__ inv,
                                                       const int64_t* __restrict__ lags, int64_t n,
                                                       float* __restrict__ h) {
  __shared__ double b[CONSTRUCT_MAX_M * (PROJECT_ROWS + 1)];
  const int64_t r0 = (int64_t)blockIdx.x * PROJECT_ROWS;
  for (int j = (int)threadIdx.x & 31; j < m; j += 32) {
    constexpr int PER = PROJECT_ROWS / 8;
    double v[PER];
#pragma unroll
    for (int a = 0; a < PER; ++a) v[a] = 0.0;
    for (int q = 0; q < segs; ++q) {
#pragma unroll
      for (int a = 0; a < PER; ++a) {  // rows past the last read the last one
        const int64_t r = r0 + (threadIdx.x >> 5) + 8 * a;
        v[a] += part[((int64_t)q * (rows + m) + (r < rows ? r : rows - 1)) * m + j];
      }
    }
#pragma unroll
    for (int a = 0; a < PER; ++a) b[j * (PROJECT_ROWS + 1) + (threadIdx.x >> 5) + 8 * a] = v[a];
  }
  __syncthreads();
  const int lane = (int)threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  if (r0 + lane >= rows) return;
  const int64_t l = lags[r0 + lane];
  const double inv_n = 1.0 / (double)n;
  for (int k = wave; k < m; k += 4) {
    double v = 0.0;
    for (int j = 0; j < m; ++j) v = fma(inv[k * m + j], b[j * (PROJECT_ROWS + 1) + lane], v);
    h[(int64_t)k * n + l] = (float)(v * inv_n);
  }
}

// In-place LU with partial pivoting of E (m x m): L unit lower, U upper,
// perm[i] = original row of pivot row i; *fail = 1 when a pivot is not above
// 1e-12 of the largest entry of E.
__global__ __launch_bounds__(256) void k_lu(double* __restrict__ E, int m, int* __restrict__ perm,
                                            int* __restrict__ fail) {
  __shared__ double S[CONSTRUCT_MAX_M * CONSTRUCT_MAX_M];
  __shared__ int pr[CONSTRUCT_MAX_M];
  __shared__ int bad, piv;
  __shared__ double emax;
  for (int i = threadIdx.x; i < m * m; i += blockDim.x) S[i] = E[i];
  for (int i = threadIdx.x; i < m; i += blockDim.x) pr[i] = i;
  __syncthreads();
  if (threadIdx.x == 0) {
    bad = 0;
    double a = 0.0;
    for (int i = 0; i < m * m; ++i) a = fmax(a, fabs(S[i]));
    emax = a;
  }
  __syncthreads();
  for (int j = 0; j < m; ++j) {
    if (threadIdx.x == 0) {
      int best = j;
      for (int i = j + 1; i < m; ++i)
        if (fabs(S[i * m + j]) > fabs(S[best * m + j])) best = i;
      if (!(fabs(S[best * m + j]) > 1e-12 * emax)) bad = 1;
      piv = best;
    }
    __syncthreads();
    if (piv != j) {
      for (int c = threadIdx.x; c < m; c += blockDim.x) {
        const double t = S[j * m + c];
        S[j * m + c] = S[piv * m + c];
        S[piv * m + c] = t;
      }
      if (threadIdx.x == 0) {
        const int t = pr[j];
        pr[j] = pr[piv];
        pr[piv] = t;
      }
    }
    __syncthreads();
    const double d = S[j * m + j];
    if (d != 0.0) {
      for (int i = j + 1 + threadIdx.x; i < m; i += blockDim.x) S[i * m + j] /= d;
      __syncthreads();
      for (int e = threadIdx.x; e < (m - j - 1) * (m - j - 1); e += blockDim.x) {
        const int i = j + 1 + e / (m - j - 1), c = j + 1 + e % (m - j - 1);
        S[i * m + c] -= S[i * m + j] * S[j * m + c];
      }
    }
    __syncthreads();
  }
  for (int i = threadIdx.x; i < m * m; i += blockDim.x) E[i] = S[i];
  for (int i = threadIdx.x; i < m; i += blockDim.x) perm[i] = pr[i];
  if (threadIdx.x == 0) *fail = bad;
}

// One thread per TVIR row r: solve E c = t in float64 in the row's slot of
// `work` (m values), starting from the row of `src`, and write
// h[k][lags[r]] = c_k / n.  F holds unit-lower L and U with the row
// permutation perm.
__global__ __launch_bounds__(256) void k_row_solve(const double* __restrict__ F, const int* __restrict__ perm, int m,
                                                   const double* __restrict__ src, double* __restrict__ work,
                                                   int64_t rows, const int64_t* __restrict__ lags, int64_t n,
                                                   float* __restrict__ h) {
  __shared__ double S[CONSTRUCT_MAX_M * CONSTRUCT_MAX_M];
  for (int i = threadIdx.x; i < m * m; i += blockDim.x) S[i] = F[i];
  __syncthreads();
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= rows) return;
  const double* a = src + r * m;
  double* b = work + r * m;
  for (int i = 0; i < m; ++i) b[i] = a[perm[i]];
  for (int i = 0; i < m; ++i) {  // L y = P t, L unit lower
    double v = b[i];
    for (int p = 0; p < i; ++p) v -= S[i * m + p] * b[p];
    b[i] = v;
  }
  for (int i = m - 1; i >= 0; --i) {  // U c = y
    double v = b[i];
    for (int p = i + 1; p < m; ++p) v -= S[i * m + p] * b[p];
    b[i] = v / S[i * m + i];
  }
  const int64_t l = lags[r];
  const double inv_n = 1.0 / (double)n;
  for (int k = 0; k < m; ++k) h[(int64_t)k * n + l] = (float)(b[k] * inv_n);
}

__global__ __launch_bounds__(256) void k_fill_zero(float* __restrict__ x, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) x[i] = 0.f;
}

// E[i][k] = W[k][nodes[i]] (float64), and the samples as float64 rows
__global__ __launch_bounds__(256) void k_node_matrix(const float* __restrict__ W, int m, int64_t n,
                                                     const int64_t* __restrict__ nodes, double* __restrict__ E) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= m * m) return;
  const int i = e / m, k = e % m;
  E[e] = (double)W[(int64_t)k * n + nodes[i]];
}

__global__ __launch_bounds__(256) void k_to_double(const float* __restrict__ x, int64_t n, double* __restrict__ y) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) y[i] = (double)x[i];
}

// out[k][l] = in[k][-l] on every axis (lag layout), 1D (n1 == 1) or 2D
__global__ __launch_bounds__(256) void k_flip(const float* __restrict__ in, float* __restrict__ out, int64_t count,
                                              int64_t n0, int64_t n1) {
  const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= count * n0 * n1) return;
  const int64_t k = g / (n0 * n1), rem = g % (n0 * n1);
  const int64_t i = rem / n1, j = rem % n1;
  out[g] = in[(k * n0 + (n0 - i) % n0) * n1 + (n1 - j) % n1];
}

static inline unsigned blocks_of(int64_t n) { return (unsigned)((n + 255) / 256); }

LaunchStatus launch_project(const float* tvir, int64_t rows, const float* windows, int m, int64_t n, double* part,
                            double* inv, int* fail, const int64_t* lags, float* h, hipStream_t s) {
  const int segs = gemm_segments(rows, m, n);
  const dim3 grid((unsigned)((rows + GEMM_ROWS - 1) / GEMM_ROWS + (m + GEMM_ROWS - 1) / GEMM_ROWS),
                  (unsigned)((m + GEMM_COLS - 1) / GEMM_COLS), (unsigned)segs);
  hipLaunchKernelGGL(k_gemm_nt_f32, grid, dim3(256), 0, s, tvir, rows, windows, m, n, gemm_seg_stages(rows, m, n),
                     part);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_gram_inverse, dim3(1), dim3(1024), 0, s, part, segs, rows, m, inv, fail);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_project_solve, dim3((unsigned)((rows + PROJECT_ROWS - 1) / PROJECT_ROWS)), dim3(256), 0, s, part,
                     segs, rows, m, inv, lags, n, h);
  return hipGetLastError();
}

LaunchStatus launch_lu(double* E, int m, int* perm, int* fail, hipStream_t s) {
  hipLaunchKernelGGL(k_lu, dim3(1), dim3(256), 0, s, E, m, perm, fail);
  return hipGetLastError();
}

LaunchStatus launch_row_solve(const double* F, const int* perm, int m, const double* src, double* work, int64_t rows,
                              const int64_t* lags, int64_t n, float* h, hipStream_t s) {
  hipLaunchKernelGGL(k_row_solve, dim3(blocks_of(rows)), dim3(256), 0, s, F, perm, m, src, work, rows, lags, n, h);
  return hipGetLastError();
}

LaunchStatus launch_fill_zero(float* x, int64_t n, hipStream_t s) {
  hipLaunchKernelGGL(k_fill_zero, dim3(blocks_of(n)), dim3(256), 0, s, x, n);
  return hipGetLastError();
}

LaunchStatus launch_node_matrix(const float* W, int m, int64_t n, const int64_t* nodes, double* E, hipStream_t s) {
  hipLaunchKernelGGL(k_node_matrix, dim3(blocks_of((int64_t)m * m)), dim3(256), 0, s, W, m, n, nodes, E);
  return hipGetLastError();
}

LaunchStatus launch_to_double(const float* x, int64_t n, double* y, hipStream_t s) {
  hipLaunchKernelGGL(k_to_double, dim3(blocks_of(n)), dim3(256), 0, s, x, n, y);
  return hipGetLastError();
}

LaunchStatus launch_flip(const float* in, float* out, int64_t count, int64_t n0, int64_t n1, hipStream_t s) {
  hipLaunchKernelGGL(k_flip, dim3(blocks_of(count * n0 * n1)), dim3(256), 0, s, in, out, count, n0, n1);
  return hipGetLastError();
}

}  // namespace pc
