// Periodic orthonormal discrete wavelet transforms for Meyer's operator
// representation (section 4.5): the TVIR is expanded in a tensor wavelet
// basis and the expansion is regrouped into windows psi_mu and responses
// c~_mu = sum_lambda c_{lambda,mu} psi_lambda, which are syntheses (inverse
// transforms) of coefficient vectors.
//
// One analysis level on a vector a of length len (periodic):
//   lo[i] = sum_k h[k] a[(2i + k) mod len],  hi[i] = sum_k g[k] a[(2i + k) mod len],
// g[k] = (-1)^k h[L - 1 - k]; coefficients in pyramid order
// [a_J, d_J, ..., d_1].  Synthesis is the transpose, evaluated as a gather:
//   a[p] = sum over k with k = p (mod 2) of h[k] lo[i] + g[k] hi[i],
//   i = ((p - k) / 2) mod (len / 2).
// Vector b's element i lives at base + b * dist + i * stride, so a 2D
// transform is a pass over rows (stride 1) and one over columns (dist 1).
#include <algorithm>
#include <mutex>

#include "pc_internal.hpp"

namespace pc {

// thread -> (vector, element): the faster-moving one is the one adjacent in
// memory, so that consecutive threads touch consecutive addresses
// (I: unsigned 32-bit where the launch's elements fit, else 64-bit)
template <class I>
__device__ __forceinline__ void split_index(I t, I count, I len, bool vec_fast, int64_t& b, int64_t& i) {
  if (vec_fast) {
    b = t % count;
    i = t / count;
  } else {
    i = t % len;
    b = t / len;
  }
}

// one analysis level: src (len elements per vector, strided) -> lo into dst
// (len/2, strided) and hi into out at positions [len/2, len) (strided);
// len is a power of two
template <class I>
__global__ __launch_bounds__(256) void k_dwt_level(const float* __restrict__ src, int64_t s_stride, int64_t s_dist,
                                                   float* __restrict__ lo_dst, int64_t l_stride, int64_t l_dist,
                                                   float* __restrict__ out, int64_t o_stride, int64_t o_dist,
                                                   int64_t count, int64_t len, WaveletFilter f, int vec_fast) {
  const int64_t half = len / 2;
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= count * half) return;
  int64_t b, i;
  split_index<I>((I)t, (I)count, (I)half, vec_fast != 0, b, i);
  const float* a = src + b * s_dist;
  float lo = 0.f, hi = 0.f;
  for (int k = 0; k < f.taps; ++k) {
    const float v = a[((2 * i + k) & (len - 1)) * s_stride];
    lo = fmaf(f.h[k], v, lo);
    hi = fmaf(f.g[k], v, hi);
  }
  lo_dst[b * l_dist + i * l_stride] = lo;
  out[b * o_dist + (half + i) * o_stride] = hi;
}

// one synthesis level: lo (strided) and hi (strided in c, positions
// [half, 2 half)) -> dst (2 half elements, strided); half is a power of two
template <class I>
__global__ __launch_bounds__(256) void k_idwt_level(const float* __restrict__ lo_src, int64_t l_stride, int64_t l_dist,
                                                    const float* __restrict__ c, int64_t c_stride, int64_t c_dist,
                                                    float* __restrict__ dst, int64_t d_stride, int64_t d_dist,
                                                    int64_t count, int64_t half, WaveletFilter f, int vec_fast) {
  const int64_t len = 2 * half;
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= count * len) return;
  int64_t b, p;
  split_index<I>((I)t, (I)count, (I)len, vec_fast != 0, b, p);
  const float* lo = lo_src + b * l_dist;
  const float* hi = c + b * c_dist + half * c_stride;
  float acc = 0.f;
  for (int k = (int)(p & 1); k < f.taps; k += 2) {
    const int64_t i = ((p - k) >> 1) & (half - 1);  // p - k is even
    acc = fmaf(f.h[k], lo[i * l_stride], acc);
    acc = fmaf(f.g[k], hi[i * c_stride], acc);
  }
  dst[b * d_dist + p * d_stride] = acc;
}

// out[b][i] = in[b][i] for i < len (strided on both sides)
__global__ __launch_bounds__(256) void k_copy_strided(const float* __restrict__ in, int64_t i_stride, int64_t i_dist,
                                                      float* __restrict__ out, int64_t o_stride, int64_t o_dist,
                                                      int64_t count, int64_t len, int vec_fast) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= count * len) return;
  int64_t b, i;
  split_index<int64_t>(t, count, len, vec_fast != 0, b, i);
  out[b * o_dist + i * o_stride] = in[b * i_dist + i * i_stride];
}

// ---------------------------------------------------------------------------
// All levels in one launch.  A workgroup takes V vectors of n samples, loads
// them into LDS once, runs every level there (one barrier per level) and
// writes each coefficient once, so the transform moves its input and its
// output and nothing else.  VF (columns of a matrix: vectors adjacent in
// memory): V neighbouring vectors, a row of the tile is V consecutive
// floats, and neighbouring tiles run on one XCD (xcd_major), whose L2 joins
// their parts of a 128-byte line.  At a few megabytes one round of
// workgroups covers the matrix, so a launch lasts as long as one workgroup's
// load, its levels one after another, and its stores.  Measured (2048 x 2048,
// 7 levels, 4 taps): rows 12.0 us and columns 14.3 us per launch, where the
// eight launches of a launch per level took 48 to 70 us; the four synchronous
// calls of both axes and directions 314 -> 122 us.
// ---------------------------------------------------------------------------
constexpr int FUSED_MAX_THREADS = 1024;

// LDS position of element i of vector v (vectors of len elements)
template <bool VF>
__device__ __forceinline__ int fpos(int v, int i, int len, int lv) {
  return VF ? (i << lv) + v : v * len + i;
}
// element t of a tile of V vectors x (1 << ll) elements
template <bool VF>
__device__ __forceinline__ void fsplit(int t, int lv, int ll, int& v, int& i) {
  if (VF) {
    v = t & ((1 << lv) - 1);
    i = t >> lv;
  } else {
    i = t & ((1 << ll) - 1);
    v = t >> ll;
  }
}

// Offset (in samples) of element i of vector v from the tile's first
// vector.  SMALL: strides below 2^24 and a tile within 2^31 bytes (the host
// checks), so two full-rate 24-bit multiplications and a 32-bit offset from
// a uniform base; the 64-bit form (six quarter-rate multiplications per
// sample) cost 12.9 us for the rows of a 2048 x 2048 matrix, this 12.0.
template <bool SMALL>
__device__ __forceinline__ auto foff(int v, int i, int64_t stride, int64_t dist) {
  if constexpr (SMALL)
    return __umul24((unsigned)v, (unsigned)dist) + __umul24((unsigned)i, (unsigned)stride);
  else
    return v * dist + i * stride;
}

// The tile's first n elements of every vector into LDS, eight loads in
// flight per thread.  Vectors past the last one read the last one; their
// results are not stored.
template <bool VF, bool SMALL>
__device__ __forceinline__ void fused_load(float* __restrict__ A, const float* __restrict__ in, int64_t stride,
                                           int64_t dist, int vmax, int ln, int lv) {
  const int total = 1 << (ln + lv), nt = (int)blockDim.x;
  int t0 = (int)threadIdx.x;
  for (; t0 + 7 * nt < total; t0 += 8 * nt) {
    float r[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      int v, i;
      fsplit<VF>(t0 + j * nt, lv, ln, v, i);
      r[j] = in[foff<SMALL>(min(v, vmax), i, stride, dist)];
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) A[t0 + j * nt] = r[j];  // the LDS position (fpos) of v and i in both layouts
  }
  for (; t0 < total; t0 += nt) {
    int v, i;
    fsplit<VF>(t0, lv, ln, v, i);
    A[t0] = in[foff<SMALL>(min(v, vmax), i, stride, dist)];
  }
}

// TAPS > 0: the filter's length, known at compile time; 0: f.taps
template <int TAPS, bool VF, bool SMALL>
__global__ __launch_bounds__(FUSED_MAX_THREADS) void k_dwt_fused(const float* __restrict__ in, int64_t s_stride,
                                                                 int64_t s_dist, float* __restrict__ out,
                                                                 int64_t o_stride, int64_t o_dist, int64_t count,
                                                                 int ln, int levels, int lv, WaveletFilter f) {
  extern __shared__ __attribute__((aligned(16))) float sm[];
  const int taps = TAPS > 0 ? TAPS : f.taps;
  const int64_t b0 = (VF ? xcd_major(blockIdx.x, gridDim.x) : (int64_t)blockIdx.x) << lv;
  const int vmax = (int)(count - 1 - b0 < (1 << lv) - 1 ? count - 1 - b0 : (1 << lv) - 1);
  float* a = sm;                          // V x n
  float* lo_dst = sm + (1 << (ln + lv));  // V x n / 2
  fused_load<VF, SMALL>(a, in + b0 * s_dist, s_stride, s_dist, vmax, ln, lv);
  out += b0 * o_dist;
  int ll = ln;
  for (int j = 0; j < levels; ++j, --ll) {
    __syncthreads();
    const int len = 1 << ll, half = len >> 1;
    const bool last = j == levels - 1;
    float* hi_out = out + half * o_stride;
    for (int t = (int)threadIdx.x; t < (half << lv); t += (int)blockDim.x) {
      int v, i;
      fsplit<VF>(t, lv, ll - 1, v, i);
      float lo = 0.f, hi = 0.f;
#pragma unroll
      for (int k = 0; k < taps; ++k) {
        const float x = a[fpos<VF>(v, (2 * i + k) & (len - 1), len, lv)];
        lo = fmaf(f.h[k], x, lo);
        hi = fmaf(f.g[k], x, hi);
      }
      if (!last) lo_dst[t] = lo;
      if (v <= vmax) {
        const auto o = foff<SMALL>(v, i, o_stride, o_dist);
        hi_out[o] = hi;
        if (last) out[o] = lo;
      }
    }
    float* x = a;
    a = lo_dst;
    lo_dst = x;
  }
}

template <int TAPS, bool VF, bool SMALL>
__global__ __launch_bounds__(FUSED_MAX_THREADS) void k_idwt_fused(const float* __restrict__ in, int64_t s_stride,
                                                                  int64_t s_dist, float* __restrict__ out,
                                                                  int64_t o_stride, int64_t o_dist, int64_t count,
                                                                  int ln, int levels, int lv, int pair_stores,
                                                                  WaveletFilter f) {
  extern __shared__ __attribute__((aligned(16))) float sm[];
  const int taps = TAPS > 0 ? TAPS : f.taps;
  const int64_t b0 = (VF ? xcd_major(blockIdx.x, gridDim.x) : (int64_t)blockIdx.x) << lv;
  const int vmax = (int)(count - 1 - b0 < (1 << lv) - 1 ? count - 1 - b0 : (1 << lv) - 1);
  const int n = 1 << ln;
  float* c = sm;                          // V x n coefficients
  float* s1 = c + (1 << (ln + lv));       // V x n / 2: levels an odd number before the last
  float* s2 = s1 + (1 << (ln + lv)) / 2;  // V x n / 4: levels an even number before it
  fused_load<VF, SMALL>(c, in + b0 * s_dist, s_stride, s_dist, vmax, ln, lv);
  out += b0 * o_dist;
  const float* lo = c;
  int lo_len = n;  // distance of the vectors of lo (rows layout)
  int lh = ln - levels;
  for (int j = 0; j < levels; ++j, ++lh) {
    __syncthreads();
    const int half = 1 << lh, len = 2 * half;
    const bool last = j == levels - 1;
    float* dst = (levels - 1 - j) & 1 ? s1 : s2;
    for (int t = (int)threadIdx.x; t < (half << lv); t += (int)blockDim.x) {
      int v, i;
      fsplit<VF>(t, lv, lh, v, i);
      // outputs 2i and 2i + 1: both read lo and hi at i - k / 2, k < taps
      float e = 0.f, o = 0.f;
#pragma unroll
      for (int k = 0; k < taps; k += 2) {
        const int q = (i - k / 2) & (half - 1);
        const float x = lo[fpos<VF>(v, q, lo_len, lv)], y = c[fpos<VF>(v, half + q, n, lv)];
        e = fmaf(f.h[k], x, e);
        e = fmaf(f.g[k], y, e);
        o = fmaf(f.h[k + 1], x, o);
        o = fmaf(f.g[k + 1], y, o);
      }
      if (!last) {
        dst[fpos<VF>(v, 2 * i, len, lv)] = e;
        dst[fpos<VF>(v, 2 * i + 1, len, lv)] = o;
      } else if (v <= vmax) {
        const auto d = foff<SMALL>(v, 2 * i, o_stride, o_dist);
        if (pair_stores) {
          *reinterpret_cast<float2*>(out + d) = make_float2(e, o);
        } else {
          out[d] = e;
          (out + o_stride)[d] = o;
        }
      }
    }
    lo = dst;
    lo_len = len;
  }
}

static inline unsigned blocks_n(int64_t n) { return (unsigned)((n + 255) / 256); }

// Split of a fused launch: vectors per workgroup (1 << lv), threads, LDS
// bytes; false when vectors of n samples do not fit.  Rows: one vector, or
// as many as make 2048 samples.  Columns: 32 of them (whole 128-byte lines)
// down to 8 while the chip gets two workgroups per CU, else 8 or 4 for one
// per CU; fewer than 4 (16 of a line's bytes) only where there are no more.
struct FusedSplit {
  int lv, threads;
  size_t lds;
};
static bool fused_split(int64_t n, int64_t count, bool vf, FusedSplit& q) {
  constexpr int64_t LDS_MAX = 120 * 1024;
  auto bytes = [n](int lv) { return (n * 7) << lv; };  // 1.75 n floats per vector
  int lv = 0;
  if (vf) {
    auto fits = [&](int l, int64_t lds, int64_t tiles) { return bytes(l) <= lds && (count >> l) >= tiles; };
    lv = 5;
    while (lv > 2 && !fits(lv, 64 * 1024, 512)) --lv;
    if (lv == 2) lv = fits(3, LDS_MAX, 256) ? 3 : 2;
    while (lv > 0 && ((int64_t)1 << (lv - 1)) >= count) --lv;
  } else {
    while (lv < 8 && (n << lv) < 2048 && ((int64_t)1 << lv) < count) ++lv;
  }
  if (n > LDS_MAX || bytes(lv) > LDS_MAX) return false;
  const int64_t e = n << lv;
  q = FusedSplit{lv, e <= 4096 ? 256 : e <= 8192 ? 512 : 1024, (size_t)std::max<int64_t>(bytes(lv), 64)};
  return true;
}

static int ilog2(int64_t n) {
  int l = 0;
  while (((int64_t)1 << l) < n) ++l;
  return l;
}

// One fused launch over vectors of n samples.
template <bool VF, bool SMALL>
static LaunchStatus run_fused(bool synthesis, int64_t n, int levels, const WaveletFilter& f, int64_t count,
                              const float* in, int64_t is, int64_t id, float* out, int64_t os, int64_t od,
                              const FusedSplit& q, hipStream_t s) {
  const dim3 grid((unsigned)((count + ((int64_t)1 << q.lv) - 1) >> q.lv)), block((unsigned)q.threads);
  const int ln = ilog2(n);
  if (!synthesis) {
#define PC_DWT(TT)                                                                                                  \
  hipLaunchKernelGGL((k_dwt_fused<TT, VF, SMALL>), grid, block, q.lds, s, in, is, id, out, os, od, count, ln, levels, \
                     q.lv, f)
    switch (f.taps) {
      case 2: PC_DWT(2); break;
      case 4: PC_DWT(4); break;
      case 6: PC_DWT(6); break;
      case 8: PC_DWT(8); break;
      default: PC_DWT(0);
    }
#undef PC_DWT
  } else {
    // outputs 2i, 2i + 1 as one 8-byte store where every such pair is 8-byte aligned
    const int pairs = os == 1 && od % 2 == 0 && reinterpret_cast<uintptr_t>(out) % 8 == 0 ? 1 : 0;
#define PC_IDWT(TT)                                                                                                  \
  hipLaunchKernelGGL((k_idwt_fused<TT, VF, SMALL>), grid, block, q.lds, s, in, is, id, out, os, od, count, ln, levels, \
                     q.lv, pairs, f)
    switch (f.taps) {
      case 2: PC_IDWT(2); break;
      case 4: PC_IDWT(4); break;
      case 6: PC_IDWT(6); break;
      case 8: PC_IDWT(8); break;
      default: PC_IDWT(0);
    }
#undef PC_IDWT
  }
  return hipGetLastError();
}

template <bool VF>
static LaunchStatus run_fused(bool synthesis, int64_t n, int levels, const WaveletFilter& f, int64_t count,
                              const float* in, int64_t is, int64_t id, float* out, int64_t os, int64_t od,
                              const FusedSplit& q, hipStream_t s) {
  constexpr int64_t ONE24 = 1 << 24, ONE29 = 1 << 29;
  auto fits = [&](int64_t st, int64_t di) {  // every offset of a tile below 2^29 samples
    return st < ONE24 && di < ONE24 && (((int64_t)1 << q.lv) - 1) * di + n * st < ONE29;
  };
  return fits(is, id) && fits(os, od) ? run_fused<VF, true>(synthesis, n, levels, f, count, in, is, id, out, os, od, q, s)
                                      : run_fused<VF, false>(synthesis, n, levels, f, count, in, is, id, out, os, od, q, s);
}

// Levels that take a launch of their own before (analysis) or after
// (synthesis) the fused ones: those of vectors too long for LDS.
static int separate_levels(int64_t n, int levels, int64_t count, bool vf) {
  FusedSplit q;
  int j = 0;
  while (j < levels && !fused_split(n >> j, count, vf, q)) ++j;
  return j;
}

int64_t wavelet_scratch(int64_t n, int levels, int64_t count, int64_t stride, int64_t dist) {
  return separate_levels(n, levels, count, dist < stride) > 0 ? count * (n / 2) : 0;
}

LaunchStatus launch_wavelet(bool synthesis, int64_t n, int levels, const WaveletFilter& f, int64_t count,
                            int64_t stride, int64_t dist, const float* in, float* out, float* s1, float* s2,
                            hipStream_t s) {
  const bool vf = dist < stride;
  hipError_t e = hipSuccess;
  if (levels == 0) {
    hipLaunchKernelGGL(k_copy_strided, dim3(blocks_n(count * n)), dim3(256), 0, s, in, stride, dist, out, stride,
                       dist, count, n, vf ? 1 : 0);
    return hipGetLastError();
  }
  const int sep = separate_levels(n, levels, count, vf);
  const bool i32 = count * n < ((int64_t)1 << 31);
  // intermediate vectors of len samples keep the caller's order in scratch
  // (columns stay adjacent)
  auto sstride = [&](int64_t) { return vf ? count : (int64_t)1; };
  auto sdist = [&](int64_t len) { return vf ? (int64_t)1 : len; };
  FusedSplit q;
  auto fused = [&](int64_t len, int lev, const float* a, int64_t as, int64_t ad, float* b, int64_t bs, int64_t bd) {
    fused_split(len, count, vf, q);
    return vf ? run_fused<true>(synthesis, len, lev, f, count, a, as, ad, b, bs, bd, q, s)
              : run_fused<false>(synthesis, len, lev, f, count, a, as, ad, b, bs, bd, q, s);
  };
  if (!synthesis) {
    // level j reads A_j (in, then s1 / s2 alternately) and writes lo to the
    // other scratch buffer, hi to out; the fused levels finish from there
    const float* src = in;
    int64_t ss = stride, sd = dist, len = n;
    for (int j = 0; j < sep && e == hipSuccess; ++j) {
      const int64_t half = len / 2;
      const bool done = j == levels - 1;  // nothing fused follows: lo is the final approximation
      float* lo = done ? out : (j % 2 == 0) ? s1 : s2;
      const int64_t ls = done ? stride : sstride(half), ld = done ? dist : sdist(half);
      if (i32)
        hipLaunchKernelGGL(k_dwt_level<uint32_t>, dim3(blocks_n(count * half)), dim3(256), 0, s, src, ss, sd, lo, ls,
                           ld, out, stride, dist, count, len, f, vf ? 1 : 0);
      else
        hipLaunchKernelGGL(k_dwt_level<int64_t>, dim3(blocks_n(count * half)), dim3(256), 0, s, src, ss, sd, lo, ls,
                           ld, out, stride, dist, count, len, f, vf ? 1 : 0);
      e = hipGetLastError();
      src = lo;
      ss = ls;
      sd = ld;
      len = half;
    }
    if (e == hipSuccess && sep < levels) e = fused(len, levels - sep, src, ss, sd, out, stride, dist);
    return e;
  }
  // synthesis: the fused levels first, then one launch per longer level;
  // the intermediate vectors alternate between s1 and s2, the last level
  // writes out
  const float* lo = in;
  int64_t ls = stride, ld = dist;
  const int64_t flen = n >> sep;  // length after the fused levels
  if (sep < levels) {
    const bool last = sep == 0;
    float* dst = last ? out : s1;
    const int64_t ds = last ? stride : sstride(flen), dd = last ? dist : sdist(flen);
    e = fused(flen, levels - sep, in, stride, dist, dst, ds, dd);
    lo = dst;
    ls = ds;
    ld = dd;
  }
  int64_t half = flen;
  for (int j = 0; j < sep && e == hipSuccess; ++j) {
    const bool last = j == sep - 1;
    float* dst = last ? out : (j % 2 == 0) ? s2 : s1;
    const int64_t ds = last ? stride : sstride(2 * half), dd = last ? dist : sdist(2 * half);
    if (i32)
      hipLaunchKernelGGL(k_idwt_level<uint32_t>, dim3(blocks_n(count * 2 * half)), dim3(256), 0, s, lo, ls, ld, in,
                         stride, dist, dst, ds, dd, count, half, f, vf ? 1 : 0);
    else
      hipLaunchKernelGGL(k_idwt_level<int64_t>, dim3(blocks_n(count * 2 * half)), dim3(256), 0, s, lo, ls, ld, in,
                         stride, dist, dst, ds, dd, count, half, f, vf ? 1 : 0);
    e = hipGetLastError();
    lo = dst;
    ls = ds;
    ld = dd;
    half *= 2;
  }
  return e;
}

// ---------------------------------------------------------------------------
// Allocation-free transforms: the two ping-pong buffers live in a fixed
// device array instead of the library's grow-only scratch.  Each device
// holds its own copy of the array; its address is looked up once per device
// (with that device current) and kept.  The array is shared by every such
// call on a device, so calls that overlap on one device race; every entry a
// level reads was written by the level before it in the same call, so
// nothing needs clearing between calls.
// ---------------------------------------------------------------------------
static __device__ __align__(256) float scratch[WAVELET_STATIC_FLOATS];

namespace {
std::mutex g_static_mu;
float* g_static_ptr[64] = {};  // per device
}  // namespace

LaunchStatus launch_wavelet_static(bool synthesis, int64_t n, int levels, const WaveletFilter& f, int64_t count,
                                   int64_t stride, int64_t dist, const float* in, float* out, hipStream_t s) {
  if (count * (n / 2) > WAVELET_STATIC_FLOATS / 2) return hipErrorInvalidValue;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
  float* base = nullptr;
  {
    std::lock_guard<std::mutex> g(g_static_mu);
    if (!g_static_ptr[dev]) {
      void* ptr = nullptr;
      e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
      if (e != hipSuccess) return e;
      g_static_ptr[dev] = static_cast<float*>(ptr);
    }
    base = g_static_ptr[dev];
  }
  float* s1 = base;
  float* s2 = base + WAVELET_STATIC_FLOATS / 2;
  return launch_wavelet(synthesis, n, levels, f, count, stride, dist, in, out, s1, s2, s);
}

}  // namespace pc
