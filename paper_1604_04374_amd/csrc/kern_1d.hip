// 1D kernels of the convolution-product expansion (eq. 1.4 and its adjoint).
//
// Real signals are processed two at a time as one complex signal
// (u_a + i u_b): windows and impulse responses are real, so
// H_m (u_a + i u_b) = H_m u_a + i H_m u_b exactly, and one complex FFT serves
// two outputs.  The identity of section 3.5 is applied once per output:
// since the DFT is linear, sum_k F(H_k . U_k) = F(sum_k H_k . U_k), so the
// forward pass pays m forward transforms and one inverse transform, and the
// adjoint pass one forward and m inverse transforms.
#include <algorithm>

#include "fft_engine.hpp"
#include "pc_internal.hpp"

namespace pc {

// The thread index, opaque to the compiler, for transforms inside a runtime
// loop: their per-element LDS addresses are recomputed instead of held in
// registers for the whole loop.
__device__ __forceinline__ int opaque1d(int x) {
  asm volatile("" : "+v"(x));
  return x;
}

#define PC_FOR_EACH_L(X) \
  X(64) X(128) X(256) X(512) X(1024) X(2048) X(4096) X(8192) \
  X(96) X(192) X(384) X(768) X(1536) X(3072) X(6144)

bool fft_size_supported(int64_t L) {
  switch (L) {
#define PC_CASE(LL) case LL:
    PC_FOR_EACH_L(PC_CASE)
#undef PC_CASE
    return true;
    default:
      return false;
  }
}

// ===========================================================================
// N <= 8192: one workgroup (or one slice of it) per signal pair
// ===========================================================================

// Plan-time spectra H_k = F^* h_k (full complex, natural order).
template <int L>
__global__ __launch_bounds__(ffts_per_block(L) * fft_threads(L)) void k_spec1d_full(
    const float* __restrict__ h, float2* __restrict__ H, int m, const float2* __restrict__ tw) {
  constexpr int P = points_per_thread(L), T = L / P, NF = ffts_per_block(L);
  __shared__ float2 lds[NF * lds_len<L>()];
  __shared__ float2 twl[L];
  stage_twiddles<L>(twl, tw);
  const int c = threadIdx.x / T, t = threadIdx.x % T;
  const int k = blockIdx.x * NF + c;
  const bool ok = k < m;
  float2 v[P];
#pragma unroll
  for (int e = 0; e < P; ++e) v[e] = make_float2(ok ? h[(int64_t)k * L + t + T * e] : 0.f, 0.f);
  fft_wg<L, P, false>(v, lds + c * lds_len<L>(), twl, t);
  if (ok) {
#pragma unroll
    for (int e = 0; e < P; ++e) H[(int64_t)k * L + t + T * e] = v[e];
  }
}

// Points per thread of the 1D kernels with no more than a pair's work in a
// workgroup.  The large batches' kernels take 16 at 4096 points, where the
// transform then needs one exchange less (390 pairs, 8 terms: 40 us at 8,
// 31 at 16); 8 are the better elsewhere (1024 points, 3 terms, 8000 pairs:
// 72 / 54 us per forward at 16 / 8; 128 points, 32 terms, 20000 pairs: 108 at
// 4, 91 at 8).
constexpr int split_points(int L) { return L % 3 == 0 ? 12 : L >= 8192 ? 16 : 8; }
constexpr int split_threads(int L) { return L / split_points(L); }
constexpr int wide_points(int L) { return L == 256 || L == 1024 || L == 2048 ? 16 : 0; }  // (0: none)
constexpr int plain_points(int L) { return L == 4096 ? 16 : split_points(L); }
constexpr int plain_threads(int L) { return L / plain_points(L); }
constexpr int plain_slots(int L) { return plain_threads(L) >= 256 ? 1 : 256 / plain_threads(L); }

// y = H_m u for signal pairs, one pair per transform slot: batches with a
// pair for every slot of the chip (k_small1d_split takes the others).
template <int L>
__global__ __launch_bounds__(plain_slots(L) * plain_threads(L)) void k_fwd1d_small(
    const float* __restrict__ u, float* __restrict__ y, int64_t batch, int m, const float* __restrict__ w,
    const float2* __restrict__ H, const float2* __restrict__ tw) {
  constexpr int P = plain_points(L), T = L / P, NF = plain_slots(L);
  __shared__ float2 lds[NF * lds_len<L>()];
  __shared__ float2 twl[L];
  stage_twiddles<L>(twl, tw);
  const int c = threadIdx.x / T, t = threadIdx.x % T;
  const int64_t pair = (int64_t)blockIdx.x * NF + c;
  const int64_t sa = 2 * pair, sb = sa + 1;
  const bool va = sa < batch, vb = sb < batch;
  float ua[P], ub[P];
#pragma unroll
  for (int e = 0; e < P; ++e) {
    const int n = t + T * e;
    ua[e] = va ? u[sa * L + n] : 0.f;
    ub[e] = vb ? u[sb * L + n] : 0.f;
  }
  float2 acc[P];
#pragma unroll
  for (int e = 0; e < P; ++e) acc[e] = make_float2(0.f, 0.f);
  float2* my = lds + c * lds_len<L>();
  for (int k = 0; k < m; ++k) {
    float2 v[P];
    const float* wk = w + (int64_t)k * L;
#pragma unroll
    for (int e = 0; e < P; ++e) {
      const float ww = wk[t + T * e];
      v[e] = make_float2(ww * ua[e], ww * ub[e]);
    }
    fft_wg<L, P, false>(v, my, twl, t);
    const float2* Hk = H + (int64_t)k * L;
#pragma unroll
    for (int e = 0; e < P; ++e) acc[e] = cfma(acc[e], Hk[t + T * e], v[e]);
  }
  fft_wg<L, P, true>(acc, my, twl, t);
  const float sc = 1.0f / (float)L;
#pragma unroll
  for (int e = 0; e < P; ++e) {
    const int n = t + T * e;
    if (va) y[sa * L + n] = acc[e].x * sc;
    if (vb) y[sb * L + n] = acc[e].y * sc;
  }
}

// x = H_m^* v for signal pairs, one pair per transform slot.  From 3072 points
// on two waves per SIMD are asked for (4200 pairs of 3072 samples, 8 terms:
// 351 us without, 280 with); shorter transforms need the waves (8000 pairs of
// 1024, 3 terms: 75 us with, 54 without).
template <int L>
__global__ __launch_bounds__(plain_slots(L) * plain_threads(L))
    __attribute__((amdgpu_waves_per_eu(1, L >= 3072 ? 2 : 8))) void k_adj1d_small(
    const float* __restrict__ vin, float* __restrict__ x, int64_t batch, int m, const float* __restrict__ w,
    const float2* __restrict__ H, const float2* __restrict__ tw) {
  constexpr int P = plain_points(L), T = L / P, NF = plain_slots(L);
  __shared__ float2 lds[NF * lds_len<L>()];
  __shared__ float2 twl[L];
  stage_twiddles<L>(twl, tw);
  const int c = threadIdx.x / T, t = threadIdx.x % T;
  const int64_t pair = (int64_t)blockIdx.x * NF + c;
  const int64_t sa = 2 * pair, sb = sa + 1;
  const bool va = sa < batch, vb = sb < batch;
  float2 V[P];
#pragma unroll
  for (int e = 0; e < P; ++e) {
    const int n = t + T * e;
    V[e] = make_float2(va ? vin[sa * L + n] : 0.f, vb ? vin[sb * L + n] : 0.f);
  }
  float2* my = lds + c * lds_len<L>();
  fft_wg<L, P, false>(V, my, twl, t);
  float2 acc[P];
#pragma unroll
  for (int e = 0; e < P; ++e) acc[e] = make_float2(0.f, 0.f);
  for (int k = 0; k < m; ++k) {
    const float2* Hk = H + (int64_t)k * L;
    float2 g[P];
#pragma unroll
    for (int e = 0; e < P; ++e) g[e] = cmulc(V[e], Hk[t + T * e]);
    fft_wg<L, P, true>(g, my, twl, t);
    const float* wk = w + (int64_t)k * L;
#pragma unroll
    for (int e = 0; e < P; ++e) {
      const float ww = wk[t + T * e];
      acc[e].x = fmaf(ww, g[e].x, acc[e].x);
      acc[e].y = fmaf(ww, g[e].y, acc[e].y);
    }
  }
  const float sc = 1.0f / (float)L;
#pragma unroll
  for (int e = 0; e < P; ++e) {
    const int n = t + T * e;
    if (va) x[sa * L + n] = acc[e].x * sc;
    if (vb) x[sb * L + n] = acc[e].y * sc;
  }
}

// The same at 16 points per thread: one exchange less per transform, and two
// workgroups per compute unit with every address in registers.  split: the NF
// slots of a workgroup share one pair, take its terms in turn and add their
// sums in LDS.  For calls that fill those workgroups' rounds (adj_wide).
// (split is an argument: the loop of a kernel without it is scheduled worse,
// 191 instead of 170 us at 4096 signals of 1024 samples, 64 terms)
template <int L>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 2))) void k_adj1d_wide(
    const float* __restrict__ vin, float* __restrict__ x, int64_t batch, int m, const float* __restrict__ w,
    const float2* __restrict__ H, const float2* __restrict__ tw, int split) {
  constexpr int P = 16, T = L / P, NF = 256 / T;
  __shared__ float2 lds[NF * lds_len<L>()];
  __shared__ float2 twl[L];
  stage_twiddles<L>(twl, tw);
  const int c = threadIdx.x / T, t = threadIdx.x % T;
  const int64_t pair = split ? (int64_t)blockIdx.x : (int64_t)blockIdx.x * NF + c;
  const int64_t sa = 2 * pair, sb = sa + 1;
  const bool va = sa < batch, vb = sb < batch;
  float2 V[P];
#pragma unroll
  for (int e = 0; e < P; ++e) {
    const int n = t + T * e;
    V[e] = make_float2(va ? vin[sa * L + n] : 0.f, vb ? vin[sb * L + n] : 0.f);
  }
  float2* my = lds + c * lds_len<L>();
  fft_wg<L, P, false>(V, my, twl, t);
  float2 acc[P];
#pragma unroll
  for (int e = 0; e < P; ++e) acc[e] = make_float2(0.f, 0.f);
  // every slot makes the same number of transform calls (they hold barriers):
  // a slot past the last term transforms a valid one with zero weight
  const int nk = split ? (m + NF - 1) / NF : m;
  for (int i = 0; i < nk; ++i) {
    const int kt = split ? c + NF * i : i;
    const int k = kt < m ? kt : m - 1;
    const float live = kt < m ? 1.f : 0.f;
    const float2* Hk = H + (int64_t)k * L;
    float2 g[P];
#pragma unroll
    for (int e = 0; e < P; ++e) g[e] = cmulc(V[e], Hk[t + T * e]);
    fft_wg<L, P, true>(g, my, twl, t);
    const float* wk = w + (int64_t)k * L;
#pragma unroll
    for (int e = 0; e < P; ++e) {
      const float ww = live * wk[t + T * e];
      acc[e].x = fmaf(ww, g[e].x, acc[e].x);
      acc[e].y = fmaf(ww, g[e].y, acc[e].y);
    }
  }
  if (split) {
    __syncthreads();  // every slot's transforms are done with LDS
#pragma unroll
    for (int e = 0; e < P; ++e) my[lpad(t + T * e)] = acc[e];
    __syncthreads();
    if (c > 0) return;
    for (int sl = 1; sl < NF; ++sl) {
#pragma unroll
      for (int e = 0; e < P; ++e) acc[e] = cadd(acc[e], lds[sl * lds_len<L>() + lpad(t + T * e)]);
    }
  }
  const float sc = 1.0f / (float)L;
#pragma unroll
  for (int e = 0; e < P; ++e) {
    const int n = t + T * e;
    if (va) x[sa * L + n] = acc[e].x * sc;
    if (vb) x[sb * L + n] = acc[e].y * sc;
  }
}

// ---------------------------------------------------------------------------
// Small batches: both directions with a pair's terms spread over the chip.
// The terms go to G workgroups per pair and, inside one, to S = 2^ls of its NF
// transform slots (the other slots take other pairs, so that none is idle);
// slot s of workgroup g takes terms g S + s, g S + s + G S, ...  By linearity
// every slot ends with its own share of the output samples (forward: its
// spectral sum transformed back; adjoint: its windowed inverses); the slots'
// shares are added in LDS, and with G > 1 the workgroups leave theirs in
// `part`, which k_small1d_sum adds in the order of g.
//
// What bounds it is latency: one transform after another.  Hence fewer
// points per thread than the throughput kernels (more wavefronts per
// transform), loads of the next term issued before the current transform,
// and wave-local exchanges where a transform fits a wavefront.  Measured (us
// per call, forward / adjoint; one workgroup per pair at the throughput
// kernels' points per thread -> here): 37 signals of 3072 samples, 12 terms,
// 61.5 / 67.1 -> 13.6 / 13.4; 64 of 8192, 30 terms, 209 / 143 -> 37.5 / 37.6;
// 1 of 8192, 8 terms, 60.9 / 44.0 -> 16.3 / 16.5.  A last-arriving workgroup
// that adds the shares instead of a second launch took 46 us where this
// takes 13.6: every workgroup's device-scope fence writes its XCD's L2 back.
// ---------------------------------------------------------------------------

template <int L, int P, int NT, bool ADJ>
__global__ __launch_bounds__(NT) void k_small1d_split(
    const float* __restrict__ u, float* __restrict__ y, int64_t batch, int m, const float* __restrict__ w,
    const float2* __restrict__ H, const float2* __restrict__ tw, int ls, int G, float2* __restrict__ part) {
  constexpr int T = L / P, NF = NT / T;
  // an exchange region per slot; at the end NF x L sums
  __shared__ float2 lds[NF * lds_len<L>()];
  __shared__ float2 twl[L];
  // forward slots of whole wavefronts: the pair's and the terms' addresses are
  // scalar (the adjoint is slower so, 8.7 and 9.0 us at 1 signal of 1024)
  const int tid = (int)threadIdx.x, t = tid % T;
  const int c = NF == 1 ? 0 : !ADJ && T % 64 == 0 ? __builtin_amdgcn_readfirstlane(tid / T) : tid / T;
  const int slot = c & ((1 << ls) - 1);  // of its pair's
  const int64_t pairs = (batch + 1) / 2;
  const int64_t pair0 = (int64_t)(blockIdx.x / G) * (NF >> ls);  // the workgroup's first
  const int64_t praw = pair0 + (c >> ls);
  const bool have = praw < pairs;
  const int64_t pair = have ? praw : pairs - 1;  // slots past the last pair run it again and store nothing
  const int g = (int)(blockIdx.x % G);
  TwStage<L, NT> ts;
  ts.load(tw, tid);
  const float* ua = u + 2 * pair * L;
  const bool vb = 2 * pair + 1 < batch;
  const float* ub = vb ? ua + L : ua;  // an odd batch's last pair reads its signal twice, the second zeroed
  float xa[P], xb[P];
#pragma unroll
  for (int e = 0; e < P; ++e) {
    xa[e] = ua[t + T * e];
    xb[e] = ub[t + T * e];
  }
  // a slot past the last term runs a valid one with zero weight (the
  // transforms may hold barriers)
  const int step = G << ls, nk = (m - (g << ls) + step - 1) / step;  // g S < m: the same count in every slot
  auto term = [&](int i) { return (g << ls) + slot + step * i; };
  // the factor that a term's transform needs first is loaded a term ahead, the
  // other one beside the transform (both a term ahead: 176 registers instead
  // of 147 at 768 points, two waves per SIMD instead of three: 42.4 and 34.3 us
  // per forward of 1030 signals, 32 terms); both at once for the first term of
  // short transforms, which cover less of a load (1 signal of 1024 samples:
  // 18.1 and 17.7 us per forward and adjoint)
  float wv[P];
  float2 hv[P];
  auto load_w = [&](int i) {
    const float* wk = w + (int64_t)(term(i) < m ? term(i) : m - 1) * L;
#pragma unroll
    for (int e = 0; e < P; ++e) wv[e] = wk[t + T * e];
  };
  auto load_h = [&](int i) {
    const float2* Hk = H + (int64_t)(term(i) < m ? term(i) : m - 1) * L;
#pragma unroll
    for (int e = 0; e < P; ++e) hv[e] = Hk[t + T * e];
  };
  constexpr bool BOTH = L <= 1024;
  if (BOTH || !ADJ) load_w(0);
  if (BOTH || ADJ) load_h(0);
  float2* my = lds + c * lds_len<L>();
  ts.commit(twl, tid);
  if (!vb) {
#pragma unroll
    for (int e = 0; e < P; ++e) xb[e] = 0.f;
  }
  float2 acc[P], V[ADJ ? P : 1];
#pragma unroll
  for (int e = 0; e < P; ++e) acc[e] = make_float2(0.f, 0.f);
  if constexpr (ADJ) {
#pragma unroll
    for (int e = 0; e < P; ++e) V[e] = make_float2(xa[e], xb[e]);
    fft_wv<L, P, false, SYNC_WAVE>(V, my, twl, t);
  }
  for (int i = 0; i < nk; ++i) {
    const float live = term(i) < m ? 1.f : 0.f;
    float2 v[P];
    if constexpr (ADJ) {
      if (!BOTH || i > 0) load_w(i);
#pragma unroll
      for (int e = 0; e < P; ++e) v[e] = cmulc(V[e], hv[e]);
      if (i + 1 < nk) load_h(i + 1);
      fft_wv<L, P, true, SYNC_WAVE>(v, my, twl, opaque1d(t));
#pragma unroll
      for (int e = 0; e < P; ++e) {
        const float ww = live * wv[e];
        acc[e].x = fmaf(ww, v[e].x, acc[e].x);
        acc[e].y = fmaf(ww, v[e].y, acc[e].y);
      }
    } else {
      if (!BOTH || i > 0) load_h(i);
#pragma unroll
      for (int e = 0; e < P; ++e) {
        const float ww = live * wv[e];
        v[e] = make_float2(ww * xa[e], ww * xb[e]);
      }
      if (i + 1 < nk) load_w(i + 1);
      fft_wv<L, P, false, SYNC_WAVE>(v, my, twl, opaque1d(t));
#pragma unroll
      for (int e = 0; e < P; ++e) acc[e] = cfma(acc[e], hv[e], v[e]);
    }
  }
  if constexpr (!ADJ) fft_wv<L, P, true, SYNC_WAVE>(acc, my, twl, t);
  const float sc = 1.0f / (float)L;
  if (NF == 1 || ls == 0) {  // (uniform over the workgroup)
    if (!have) return;
    if (G == 1) {
      float* ya = y + 2 * pair * L;
      float* yb = ya + L;
#pragma unroll
      for (int e = 0; e < P; ++e) {
        ya[t + T * e] = acc[e].x * sc;
        if (vb) yb[t + T * e] = acc[e].y * sc;
      }
      return;
    }
    float2* mine = part + (pair * G + g) * L;
#pragma unroll
    for (int e = 0; e < P; ++e) mine[t + T * e] = acc[e];
  } else {
    __syncthreads();  // every slot is done with its exchange region
#pragma unroll
    for (int e = 0; e < P; ++e) lds[c * L + t + T * e] = acc[e];
    __syncthreads();
    auto put = [&](int64_t pr, int n, float2 a) {
      if (G == 1) {
        y[2 * pr * L + n] = a.x * sc;
        if (2 * pr + 1 < batch) y[(2 * pr + 1) * L + n] = a.y * sc;
      } else {
        part[(pr * G + g) * L + n] = a;
      }
    };
    if (1 << ls == NF) {  // one pair
      for (int n = tid; n < L; n += NT) {
        float2 a = lds[n];
#pragma unroll
        for (int q = 1; q < NF; ++q) a = cadd(a, lds[q * L + n]);
        put(pair0, n, a);
      }
      return;
    }
    for (int i = tid; i < (NF >> ls) * L; i += NT) {
      const int pl = i / L, n = i % L;
      const int64_t pr = pair0 + pl;
      if (pr >= pairs) return;
      const float2* sh = lds + (pl << ls) * L + n;
      float2 a = cadd(sh[0], sh[L]);
#pragma unroll 2
      for (int q = 2; q < 1 << ls; q += 2) a = cadd(cadd(a, sh[q * L]), sh[(q + 1) * L]);
      put(pr, n, a);
    }
  }
}

// y = the sum of a pair's G shares, scaled, in the order of g.
template <int L>
__global__ __launch_bounds__(256) void k_small1d_sum(const float2* __restrict__ part, int G, float* __restrict__ y,
                                                     int64_t batch) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t pair = i / L;
  const int n = (int)(i % L);
  if (2 * pair >= batch) return;
  const float2* s = part + pair * G * L + n;
  float2 a = s[0];
#pragma unroll 8
  for (int g = 1; g < G; ++g) a = cadd(a, s[(int64_t)g * L]);
  const float sc = 1.0f / (float)L;
  y[2 * pair * L + n] = a.x * sc;
  if (2 * pair + 1 < batch) y[(2 * pair + 1) * L + n] = a.y * sc;
}

template <int L>
static LaunchStatus spec1d_full_t(const float* h, float2* H, int m, const float2* tw, hipStream_t s) {
  constexpr int NF = ffts_per_block(L), T = fft_threads(L);
  const int blocks = (m + NF - 1) / NF;
  hipLaunchKernelGGL(k_spec1d_full<L>, dim3(blocks), dim3(NF * T), 0, s, h, H, m, tw);
  return hipGetLastError();
}

// How a call spreads a pair's terms: workgroups per pair (0: the kernels with
// a pair per transform slot), the log2 of its slots per workgroup, and threads
// per workgroup: the split with the least expected time, of the slots and
// workgroups that leave no slot without a term.  Expected are
//   transforms one after another x (latency of their passes, which grows with
//   the points per thread, x rounds of resident workgroups + the work of a
//   compute unit, mostly the fullest's)
//   + with several workgroups, the second launch and its shares;
// the constants (us) are a least-squares fit to 39,000 timings of 64 to 8192
// samples, 1 to 32 terms and 1 to 4200 pairs, over which the choice is 1% off
// the fastest split on average.  (One pair's slots per workgroup of 512 threads
// up to 1024 points, and as many workgroups as compute units, were 10%
// further off; us per forward, so and here: 4200 signals of 192 samples, 8
// terms, 49.6 and 11.6; 1030 of 768, 3 terms, 22.4 and 10.2; 16000 of 96, 16
// terms, 178 and 21.8; 520 of 2048, 32 terms, 77.0 and 49.3.)
// From a workgroup per compute unit on (two at 2048 points) the kernels with a
// pair per slot run unless a split is expected to gain 15%: they hold less
// (1030 signals of 1024 samples, 3 terms: 10.0 us, the best split 10.8), but
// leave the chip at one wavefront per SIMD there (1030 of 3072, 16 terms: 86,
// four workgroups per pair 54).
// While the terms of a slot are few and short there is one workgroup per
// pair: the second launch costs the host as much again (1 signal of 1024
// samples, 8 terms, two per slot: 8.5 us, spread 9.7; 12 terms, three per
// slot: 11.2, spread 9.9).
// At 1024 points and 8 terms or more a pair per compute unit runs four
// transforms of 16 points per thread, a wavefront each and one exchange less
// (threads 0; us per forward, 8 and 16 points per thread: 520 signals, 32 terms
// 35.3 and 31.2, 16 terms 21.1 and 19.1; 260 signals, 16 terms 14.7 and 14.8;
// 1030 signals, 16 terms 27.1 and 29.2; 520 signals, 5 terms 11.0 and 13.1).
struct SmallSplit {
  int groups, ls, threads;
};
template <int L>
constexpr int split_threads_least() {
  return split_threads(L) > 256 ? split_threads(L) : 256;
}
template <int L>
constexpr int split_threads_most() {
  return L <= 1024 ? 512 : split_threads_least<L>();
}
template <int L>
static SmallSplit small_split_t(int m, int64_t pairs) {
  constexpr int P = split_points(L), T = L / P, CUS = 256, NF = plain_slots(L);
  constexpr double latency = make_sched(L, P).n * P * (T > 64 ? 0.04 : 0.025);
  double log2L = 0;
  for (int x = 1; x < L; x *= 2) log2L += 1;
  SmallSplit best{};
  double least = 0, one_slot = 0;  // expected: the best split's, and of one slot per pair
  auto consider = [&](int ls, int groups, int threads) {
    const int64_t per_wg = threads / T >> ls, blocks = (pairs + per_wg - 1) / per_wg * groups;
    const int lds = (threads / T * lds_len<L>() + L) * (int)sizeof(float2);
    const int waves = P == 8 ? 4 : P == 12 ? 3 : 2;  // per SIMD, of the kernel's registers
    const int64_t full = (blocks + CUS - 1) / CUS;
    const int64_t resident = std::max(1, std::min(160 * 1024 / lds, waves * 256 / threads));
    // workgroups per compute unit, mostly the fullest's
    const double load = full <= 2 ? (double)full : 0.25 * (double)blocks / CUS + 0.75 * (double)full;
    const int64_t terms = (m + ((int64_t)groups << ls) - 1) / ((int64_t)groups << ls);
    double us = (double)(terms + 1) * (latency * (double)((full + resident - 1) / resident) +
                                       0.008 * load * (threads / 256) * P * log2L);
    if (groups > 1) us += 2.0 + 5e-6 * (double)(pairs * groups) * L;
    if (ls == 0 && groups == 1 && (one_slot == 0 || us < one_slot)) one_slot = us;
    if (best.groups == 0 || us < least) {
      best = SmallSplit{groups, ls, threads};
      least = us;
    }
  };
  constexpr int MOST = split_threads_most<L>();
  const bool few = (int64_t)((m + MOST / T - 1) / (MOST / T)) * L <= 2048;
  for (int threads = split_threads_least<L>(); threads <= MOST; threads *= 2) {
    int ls = 0;
    consider(0, 1, threads);
    while ((2 << ls) <= threads / T && (1 << ls) < m) consider(++ls, 1, threads);
    const int terms = (m + (1 << ls) - 1) >> ls;  // of a slot of a single workgroup
    for (int per = 1; !few && per < terms; per += std::max(1, per / 2)) {
      const int groups = (terms + per - 1) / per;  // the fewest with that many terms per slot
      if (pairs * groups <= SMALL1D_SHARES) consider(ls, groups, threads);
    }
  }
  if ((pairs + NF - 1) / NF >= (L == 2048 ? 2 * CUS : CUS) && least > 0.85 * one_slot) return SmallSplit{0, 0, 0};
  if (L == 1024 && m >= 8 && 4 * pairs >= 3 * CUS && pairs < 2 * CUS) return SmallSplit{1, 2, 0};
  return best;
}

int small1d_groups(int L, int m, int64_t pairs) {
  switch (L) {
#define PC_CASE(LL) \
  case LL:          \
    return small_split_t<LL>(m, pairs).groups;
    PC_FOR_EACH_L(PC_CASE)
#undef PC_CASE
  }
  return 0;
}

// Whether an adjoint call takes k_adj1d_wide, whose 512 resident workgroups
// it has to fill: a pair per slot from 256 workgroups on, a pair per workgroup
// below (us per adjoint, without it and with: a pair per slot, 4096 signals of
// 1024 samples, 64 terms 192 and 170, 2600 of them 154 and 171; 2000 of 2048,
// 32 terms 107 and 94, 1300 of them 88 and 94, 4096 of them 198 and 188, of 16
// terms the same; 16384 of 256, 16 terms 41.3 and 37.6, 8192 of them 26 and
// 35, 14297 of 24 terms 57 and 52; a pair per workgroup, 774 of 2048, 32 terms
// 66 and 50, 520 of them, 64 terms 84 and 91, 366 of them, 8 terms 17.9 and
// 17.1, 16 terms 24.4 and 27.4; 640 of 1024, 64 terms 54.6 and 49.2, 8 terms
// 12.2 and 12.7; 1600 of them, 64 terms 109 and 97, 16 terms 33 and 34).  At
// 512 points 8 per thread win throughout.
template <int L>
static bool adj_wide(int m, int64_t pairs, bool& split) {
  constexpr int NF = 256 * 16 / L;
  const int64_t slots = (pairs + NF - 1) / NF;
  split = slots < 256;
  if (!split)
    return (slots <= 512 && slots >= (L == 256 ? 416 : 384)) ||
           (L == 2048 && m >= 32 && slots <= 1024 && slots >= 960);
  if (L == 1024) return (m >= 16 && pairs > 256 && pairs <= 512) || (m >= 32 && pairs > 768);
  if (L == 2048) return m >= 8 && pairs > (m <= 12 ? 176 : 256) && (m < 32 || pairs >= 384);
  return false;
}

int small1d_split_points(int L) { return split_points(L); }
int small1d_wide_points(int L) { return wide_points(L); }

template <int L, bool ADJ>
static LaunchStatus small1d_t(const Small1D& p, const float* u, float* y, int64_t batch, hipStream_t s, Tracer* tr) {
  const int64_t pairs = (batch + 1) / 2;
  if constexpr (ADJ && wide_points(L) > 0) {
    bool split = false;
    if (adj_wide<L>(p.m, pairs, split)) {
      constexpr int NF = 256 * 16 / L;
      TraceScope ts(tr, "adj1d_small", s);
      const int64_t blocks = split ? pairs : (pairs + NF - 1) / NF;
      hipLaunchKernelGGL(k_adj1d_wide<L>, dim3((unsigned)blocks), dim3(256), 0, s, u, y, batch, p.m, p.w, p.H, p.tww,
                         split ? 1 : 0);
      return hipGetLastError();
    }
  }
  const SmallSplit q = small_split_t<L>(p.m, pairs);
  if (q.groups > 0) {
    {
      TraceScope ts(tr, ADJ ? "adj1d_small" : "fwd1d_small", s);
      constexpr int WP = L == 1024 ? wide_points(L) : split_points(L), WT = split_threads_least<L>();
      const int threads = q.threads > 0 ? q.threads : WT, T = q.threads > 0 ? split_threads(L) : L / WP;
      const int64_t per_wg = threads / T >> q.ls;
      const dim3 grid((unsigned)((pairs + per_wg - 1) / per_wg * q.groups)), block(threads);
      if (q.threads == 0)
        hipLaunchKernelGGL((k_small1d_split<L, WP, WT, ADJ>), grid, block, 0, s, u, y, batch, p.m, p.w, p.H, p.tww,
                           q.ls, q.groups, p.part);
      else if (q.threads == split_threads_least<L>())
        hipLaunchKernelGGL((k_small1d_split<L, split_points(L), split_threads_least<L>(), ADJ>), grid, block, 0, s, u,
                           y, batch, p.m, p.w, p.H, p.tws, q.ls, q.groups, p.part);
      else
        hipLaunchKernelGGL((k_small1d_split<L, split_points(L), split_threads_most<L>(), ADJ>), grid, block, 0, s, u,
                           y, batch, p.m, p.w, p.H, p.tws, q.ls, q.groups, p.part);
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess || q.groups == 1) return e;
    TraceScope ts(tr, "sum1d_small", s);
    hipLaunchKernelGGL(k_small1d_sum<L>, dim3((unsigned)((pairs * L + 255) / 256)), dim3(256), 0, s, p.part, q.groups,
                       y, batch);
    return hipGetLastError();
  }
  TraceScope ts(tr, ADJ ? "adj1d_small" : "fwd1d_small", s);
  constexpr int NF = plain_slots(L);
  const dim3 grid((unsigned)((pairs + NF - 1) / NF)), block(NF * plain_threads(L));
  const float2* tw = plain_points(L) == split_points(L) ? p.tws : p.tw;
  if constexpr (ADJ)
    hipLaunchKernelGGL(k_adj1d_small<L>, grid, block, 0, s, u, y, batch, p.m, p.w, p.H, tw);
  else
    hipLaunchKernelGGL(k_fwd1d_small<L>, grid, block, 0, s, u, y, batch, p.m, p.w, p.H, tw);
  return hipGetLastError();
}

LaunchStatus launch_spec1d_full(int L, const float* h, float2* H, int m, const float2* tw, hipStream_t s) {
  switch (L) {
#define PC_CASE(LL) \
  case LL:          \
    return spec1d_full_t<LL>(h, H, m, tw, s);
    PC_FOR_EACH_L(PC_CASE)
#undef PC_CASE
  }
  return hipErrorInvalidValue;
}

LaunchStatus launch_fwd1d_small(const Small1D& p, const float* u, float* y, int64_t batch, hipStream_t s,
                                Tracer* tr) {
  switch (p.L) {
#define PC_CASE(LL) \
  case LL:          \
    return small1d_t<LL, false>(p, u, y, batch, s, tr);
    PC_FOR_EACH_L(PC_CASE)
#undef PC_CASE
  }
  return hipErrorInvalidValue;
}

LaunchStatus launch_adj1d_small(const Small1D& p, const float* v, float* x, int64_t batch, hipStream_t s,
                                Tracer* tr) {
  switch (p.L) {
#define PC_CASE(LL) \
  case LL:          \
    return small1d_t<LL, true>(p, v, x, batch, s, tr);
    PC_FOR_EACH_L(PC_CASE)
#undef PC_CASE
  }
  return hipErrorInvalidValue;
}

// ===========================================================================
// N = R * L: four-step split n = n2 + L n1, f = f1 + R f2
//
//   X[f1 + R f2] = FFT_L(a^{f1})[f2],
//   a^{f1}[n2]   = W_N^{f1 n2} sum_{n1} x[n2 + L n1] W_R^{f1 n1},
//
// with W_M = exp(-2 i pi / M).  The inverse runs the same split backwards:
//   y[n2 + L n1] = (1/N) sum_{f1} W_R^{-f1 n1} W_N^{-f1 n2} b^{f1}[n2],
//   b^{f1} = unnormalised inverse FFT_L of the class-f1 spectrum.
//
// A windowed term z = w_k . u with support [o, o + S) is transformed from its
// own origin: with z'[d] = z[o + d],
//   Z[f] = W_N^{f o} sum_d z'[d] W_N^{f d},
// so the fold reads the support contiguously (d = slot index) and the phase
// W_N^{f o} is carried by the stored spectra, Hd[k][f1][f2] =
// H_k[f] W_N^{f o_k} with f = f1 + R f2.  The adjoint uses the same frame:
// conj(Hd_k) already carries the phase W_N^{-f o_k} that restricting the
// inverse transform to the window needs.
// W_N^{f1 d} comes from the class table twC[f1 * L + d] (coalesced in d);
// W_R^{j} = twN[j * L].
// ===========================================================================

// LDS pad period of the four-step kernels' exchanges
constexpr int FPAD = 32;

// LDS exchange buffers of the four-step transform kernels.  Workgroups of 512
// or more threads use two, with ping-pong exchanges (at the register counts of
// these kernels such a workgroup is alone on its compute unit, so the second
// buffer costs no occupancy); smaller workgroups use one.
template <int L, int P>
constexpr bool fs_pingpong() {
  return L / P >= 512 || 2 * lds_len<L, FPAD>() * 8 <= 80 * 1024;
}
template <int L, int P>
constexpr int fs_lds_len() {
  return (fs_pingpong<L, P>() ? 2 : 1) * lds_len<L, FPAD>();
}
template <int L, int P>
struct FsLds {
  float2* buf[2];
  __device__ explicit FsLds(float2* lds) : buf{lds, fs_pingpong<L, P>() ? lds + lds_len<L, FPAD>() : lds} {}
  // one transform with the thread's register twiddles
  template <bool INV, int NT>
  __device__ __forceinline__ void fft(float2 (&v)[P], const float2 (&twr)[NT], int t) {
    if constexpr (fs_pingpong<L, P>()) {
      fft_wg_reg_pp<L, P, INV, FPAD>(v, buf, twr, t);
      if constexpr (fft_exchanges<L, P>() % 2 == 1) {
        float2* x = buf[0];
        buf[0] = buf[1];
        buf[1] = x;
      }
    } else {
      fft_wg_reg<L, P, INV, FPAD>(v, buf[0], twr, t);
    }
  }
};

template <int L, int R>
__device__ __forceinline__ float2 unit_root_R(const float2* __restrict__ twN, int j) {
  return twN[(j % R) * L];
}

// Load base[i] through a 32-bit unsigned byte offset from a uniform base, so
// that the address is one SGPR pair plus one VGPR (no 64-bit arithmetic).
template <class X>
__device__ __forceinline__ X ldu(const X* __restrict__ base, uint32_t i) {
  return *reinterpret_cast<const X*>(reinterpret_cast<const char*>(base) + i * (uint32_t)sizeof(X));
}

// Every L-long block that the four-step kernels pass between launches (class
// spectra Hd and Vws, class outputs Bws, gradient partials E, the modulated
// windows cw) keeps element f2 = t + T e at block_pos(f2, T) (T = L / P):
// the thread that holds f2 in the workgroup transform moves elements e and
// e + 1 with one 16-byte access, and a wave's access covers 1 KiB
// contiguously.
template <int L, int P>
__device__ __forceinline__ int block_elem(int j) {  // inverse of block_pos
  constexpr int T = L / P;
  const int blk = j / (2 * T), r = j % (2 * T);
  return (r >> 1) + T * (2 * blk + (r & 1));
}

template <int L, int P>
__device__ __forceinline__ void load_blk(const float2* __restrict__ b, float2 (&v)[P], int t) {
  static_assert(P % 2 == 0, "even points per thread");
  constexpr int T = L / P;
  const float4* b4 = reinterpret_cast<const float4*>(b);
#pragma unroll
  for (int h = 0; h < P / 2; ++h) {
    const float4 q = ldu(b4, (uint32_t)(h * T + t));
    v[2 * h] = make_float2(q.x, q.y);
    v[2 * h + 1] = make_float2(q.z, q.w);
  }
}

template <int L, int P>
__device__ __forceinline__ void store_blk(float2* __restrict__ b, const float2 (&v)[P], int t) {
  constexpr int T = L / P;
  float4* b4 = reinterpret_cast<float4*>(b);
#pragma unroll
  for (int h = 0; h < P / 2; ++h)
    b4[h * T + t] = make_float4(v[2 * h].x, v[2 * h].y, v[2 * h + 1].x, v[2 * h + 1].y);
}

// (o + d) mod N for o < N, d < N
template <uint32_t N>
__device__ __forceinline__ uint32_t wrapN(uint32_t n) {
  if constexpr ((N & (N - 1)) == 0)
    return n & (N - 1);
  else
    return min(n, n - N);  // n - N wraps above n when n < N
}

// a^{f1}[d] = sum_{c < C} cw_k^{f1,c}[d] z[o + c L + d] with
// cw_k^{f1,c}[d] = w_k[o + c L + d] W_N^{f1 (c L + d)}, for a windowed term
// whose support [o, o + S) is at most C L long (cw is zero beyond S; C is 1
// or 2, and C L <= N).  The chunk c of cw starts at cwb + c L.  All loads are
// issued before any is used.
template <int L, int R, int P, int C>
__device__ __forceinline__ void fold_short(float2 (&v)[P], int t, const float* __restrict__ xa,
                                           const float* __restrict__ xb, int o,
                                           const float2* __restrict__ cwb) {
  static_assert(C == 1 || C == 2, "one or two chunks");
  constexpr int T = L / P;
  constexpr uint32_t N = (uint32_t)L * R;
  float ra[C][P], rb[C][P];
  float2 rc[C][P];
#pragma unroll
  for (int c = 0; c < C; ++c) {
#pragma unroll
    for (int e = 0; e < P; ++e) {
      const uint32_t n = wrapN<N>((uint32_t)o + (uint32_t)(c * L + t + T * e));  // o < N, c L + d < N
      ra[c][e] = ldu(xa, n);
      rb[c][e] = ldu(xb, n);
    }
  }
#pragma unroll
  for (int c = 0; c < C; ++c) load_blk<L, P>(cwb + c * L, rc[c], t);
#pragma unroll
  for (int e = 0; e < P; ++e) {
    float2 a = cmul(make_float2(ra[0][e], rb[0][e]), rc[0][e]);
#pragma unroll
    for (int c = 1; c < C; ++c) a = cfma(a, make_float2(ra[c][e], rb[c][e]), rc[c][e]);
    v[e] = a;
  }
}

// Same for supports longer than L: a^{f1}[d] = W_N^{f1 d} sum_c z[o + d + c L] W_R^{f1 c}.
template <int L, int R, int P>
__device__ __forceinline__ void fold_long(float2 (&v)[P], int t, int f1, const float* __restrict__ xa,
                                          const float* __restrict__ xb, const float* __restrict__ wc,
                                          int o, int S, const float2* __restrict__ twC,
                                          const float2* __restrict__ twN) {
  constexpr int T = L / P;
  constexpr uint32_t N = (uint32_t)L * R;
#pragma unroll
  for (int e = 0; e < P; ++e) {
    const int d0 = t + T * e;
    float2 a = make_float2(0.f, 0.f);
    int c = 0;
    for (int d = d0; d < S; d += L, ++c) {
      const uint32_t n = wrapN<N>((uint32_t)(o + d));
      const float ww = ldu(wc, (uint32_t)d);
      const float2 z = make_float2(ww * ldu(xa, n), ww * ldu(xb, n));
      a = cfma(a, z, unit_root_R<L, R>(twN, f1 * c));
    }
    v[e] = cmul(a, ldu(twC, (uint32_t)(f1 * L + d0)));
  }
}

// Class spectra of whole signals: out[(sig*R + f1)*L + f2] = X_sig[f1 + R f2].
// pairs = true packs signals (2i, 2i+1) as one complex signal.
template <int L, int R, int P>
__global__ __launch_bounds__(L / P) void k_fold_fft(const float* __restrict__ x, int64_t n_sig, bool pairs,
                                                             float2* __restrict__ out, const float2* __restrict__ tw,
                                                             const float2* __restrict__ twC,
                                                             const float2* __restrict__ twN,
                                                             const float* __restrict__ zeros) {
  constexpr int T = L / P, N = L * R;
  // one transform per workgroup: the twiddles are read from the (cached)
  // global table rather than staged, which also leaves room for two
  // workgroups per CU
  __shared__ float2 lds[lds_len<L, FPAD>()];
  const int t = threadIdx.x;
  // the R class workgroups of a signal (pair) each read the whole signal:
  // numbered so that they run on one XCD and the signal is fetched once
  const int64_t b = xcd_major(blockIdx.x, gridDim.x);
  const int f1 = (int)(b % R);
  const int64_t idx = b / R;
  // the imaginary part: the pair's second signal, or N zeros (no pair)
  const float* xa;
  const float* xb = zeros;
  if (pairs) {
    xa = x + 2 * idx * N;
    if (2 * idx + 1 < n_sig) xb = xa + N;
  } else {
    xa = x + idx * N;
  }
  float2 wr[R];
#pragma unroll
  for (int n1 = 0; n1 < R; ++n1) wr[n1] = unit_root_R<L, R>(twN, f1 * n1);
  const float2* tc = twC + f1 * L;
  float2 v[P];
#pragma unroll
  for (int e = 0; e < P; ++e) {
    const int n2 = t + T * e;
    float2 a = make_float2(0.f, 0.f);
#pragma unroll
    for (int n1 = 0; n1 < R; ++n1) {
      const float2 z = make_float2(xa[n2 + L * n1], xb[n2 + L * n1]);
      a = cfma(a, z, wr[n1]);
    }
    v[e] = cmul(a, tc[n2]);
  }
  fft_wg<L, P, false, FPAD>(v, lds, tw, t);
  store_blk<L, P>(out + (idx * R + f1) * L, v, t);
}

// Forward, class f1 of one signal pair: sum_k Hd_k^{f1} . FFT_L(fold(w_k u)),
// then the class's inverse FFT_L, stored for the combine step.
// C: chunks of the short-support path (1 or 2; the plan's cw table), 0 for
// the long-support path.
// G term groups: workgroup (pair, f1, g) takes the terms [m g / G, m (g + 1) / G)
// and leaves its own inverse transform in slice g of Bws (k_combine1d adds
// the slices), so that a few signals still fill the chip.
// (SPLIT: G > 1; without it the group arithmetic folds away)
template <int L, int R, int P, int C, bool SPLIT>
__global__ __launch_bounds__(L / P) void k_fwd1d_large(const float* __restrict__ u, int64_t batch, Large1D p, int G) {
  constexpr int N = L * R;
  __shared__ float2 lds[fs_lds_len<L, P>()];
  FsLds<L, P> xl(lds);
  const int t = threadIdx.x;
  // the thread's twiddles stay in registers for all m + 1 transforms
  float2 twr[tw_reg_count<L, P>()];
  load_tw_reg<L, P>(twr, p.tw, t);
  const int f1 = blockIdx.x % R;
  const int64_t pg = blockIdx.x / R;  // pair G + g
  const int64_t pair = SPLIT ? pg / G : pg;
  const int g = SPLIT ? (int)(pg % G) : 0;
  const int k0 = SPLIT ? p.m * g / G : 0, k1 = SPLIT ? p.m * (g + 1) / G : p.m;
  const float* xa = u + 2 * pair * N;
  const float* xb = 2 * pair + 1 < batch ? xa + N : p.zeros;  // odd batch: a zero second signal
  float2 acc[P];
#pragma unroll
  for (int e = 0; e < P; ++e) acc[e] = make_float2(0.f, 0.f);
  for (int k = k0; k < k1; ++k) {
    const int S = p.w_len[k];
    if (S == 0) continue;
    const int o = p.w_off[k];
    const float* wc = p.wc + p.w_base[k];
    (void)wc;
    float2 v[P];
    if constexpr (C > 0)
      fold_short<L, R, P, C>(v, t, xa, xb, o, p.cw + ((int64_t)k * R + f1) * C * L);
    else
      fold_long<L, R, P>(v, t, f1, xa, xb, wc, o, S, p.twC, p.twN);
    // the spectrum loads are issued before the transform so that their
    // latency overlaps it
    float2 hv[P];
    load_blk<L, P>(p.Hd + ((int64_t)k * R + f1) * L, hv, t);
    xl.template fft<false>(v, twr, t);
#pragma unroll
    for (int e = 0; e < P; ++e) acc[e] = cfma(acc[e], hv[e], v[e]);
  }
  xl.template fft<true>(acc, twr, t);
  store_blk<L, P>(p.Bws + (pg * R + f1) * L, acc, t);
}

// y[n2 + L n1] = (1/N) sum_f1 W_R^{-f1 n1} (W_N^{-f1 n2} b^{f1}[n2]), b the
// sum of the G slices of the forward pass.
// One thread per 16-byte pair of a block (block_pos: elements n2 = t + T e
// and n2 + T, e even), so every class block is read with coalesced 16-byte
// loads.
template <int L, int R, int P, bool SPLIT>
__global__ __launch_bounds__(256) void k_combine1d(const float2* __restrict__ Bws, float* __restrict__ y, int64_t batch,
                                                   const float2* __restrict__ twC, int G) {
  constexpr int N = L * R, T = L / P;
  const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t pairs = (batch + 1) / 2;
  if (gid >= pairs * (L / 2)) return;
  const int64_t pair = gid / (L / 2);
  const int q = (int)(gid % (L / 2));  // float4 index inside a block: h T + t
  const int h = q / T, t = q % T;
  const int n2[2] = {t + T * 2 * h, t + T * (2 * h + 1)};
  float2 b[2][R];
#pragma unroll
  for (int f1 = 0; f1 < R; ++f1) {
    const float4* s = reinterpret_cast<const float4*>(Bws + (pair * (SPLIT ? G : 1) * R + f1) * L) + q;
    float4 v = s[0];
    if constexpr (SPLIT) {
      // four loads in flight (one signal of 65536 samples, 31 slices: 141 us per forward with one, 78 so)
#pragma unroll 4
      for (int g = 1; g < G; ++g) {
        const float4 a = s[(int64_t)g * (R * L / 2)];
        v = make_float4(v.x + a.x, v.y + a.y, v.z + a.z, v.w + a.w);
      }
    }
    b[0][f1] = cmulc(make_float2(v.x, v.y), twC[f1 * L + n2[0]]);
    b[1][f1] = cmulc(make_float2(v.z, v.w), twC[f1 * L + n2[1]]);
  }
  const float sc = 1.0f / (float)N;
  const int64_t sa = 2 * pair, sb = sa + 1;
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    dftR<R, true>(b[j]);
#pragma unroll
    for (int n1 = 0; n1 < R; ++n1) y[sa * N + n2[j] + L * n1] = b[j][n1].x * sc;
    if (sb < batch) {
#pragma unroll
      for (int n1 = 0; n1 < R; ++n1) y[sb * N + n2[j] + L * n1] = b[j][n1].y * sc;
    }
  }
}

// Adjoint, one item of one signal pair: g = F(conj(H_k) . V) on the item's
// samples, assembled class by class, times the window; stored for the
// overlap-add.  Long-support plans (C = 0) have one item per chunk of at most
// L samples of a term's support.  Short-support plans (C = 1 or 2) have one
// item per term, whose support is at most C L long: the R class transforms
// serve all its chunks, and each chunk takes its window and class modulation
// together from cw.
// G class groups (G divides R): workgroup (pair, item, g) takes R / G classes
// and leaves its sum in slice g of the pair's block (k_ola1d adds them).
template <int L, int R, int P, int C, bool SPLIT>
__global__ __launch_bounds__(L / P) void k_adj1d_large(Large1D p, int G) {
  constexpr int T = L / P;
  __shared__ float2 lds[fs_lds_len<L, P>()];
  FsLds<L, P> xl(lds);
  const int t = threadIdx.x;
  // the thread's twiddles stay in registers for all R transforms
  float2 twr[tw_reg_count<L, P>()];
  load_tw_reg<L, P>(twr, p.tw, t);
  const int item = blockIdx.x % p.n_items;
  const int64_t pg = blockIdx.x / p.n_items;  // pair G + g
  const int64_t pair = SPLIT ? pg / G : pg;
  const int f1_0 = SPLIT ? (int)(pg % G) * (R / G) : 0, f1_1 = SPLIT ? f1_0 + R / G : R;
  const int k = p.item_k[item];
  const int c0 = p.item_d0[item];
  const int Sc = p.item_len[item];
  const int chunk = c0 / L;  // long path: chunks start at multiples of L inside the support
  constexpr int NC = C > 0 ? C : 1;  // accumulators (chunks) per item
  float2 acc[NC][P];
#pragma unroll
  for (int c = 0; c < NC; ++c)
#pragma unroll
    for (int e = 0; e < P; ++e) acc[c][e] = make_float2(0.f, 0.f);
  const float2* Hk = p.Hd + (int64_t)k * R * L;
  const float2* Vp = p.Vws + pair * R * L;
  auto load = [&](float2(&vv)[P], float2(&hh)[P], int f1) {
    load_blk<L, P>(Vp + f1 * L, vv, t);
    load_blk<L, P>(Hk + f1 * L, hh, t);
  };
  auto prod = [&](float2(&vv)[P], const float2(&hh)[P]) {
#pragma unroll
    for (int e = 0; e < P; ++e) vv[e] = cmulc(vv[e], hh[e]);
  };
  // class f1: inverse FFT_L of conj(Hd) . V, back-modulated by W_N^{-f1 d}
  // (chunks after the first also carry W_R^{-f1 chunk}) and summed
  auto step = [&](float2(&vv)[P], int f1) {
    xl.template fft<true>(vv, twr, t);
    if constexpr (C > 0) {
      // chunk c: conj(cw_k^{f1,c}) carries W_N^{-f1 (c L + d)} and the window
#pragma unroll
      for (int c = 0; c < C; ++c) {
        float2 rt[P];
        load_blk<L, P>(p.cw + (((int64_t)k * R + f1) * C + c) * L, rt, t);
        // slots at or beyond Sc accumulate values that are never stored
#pragma unroll
        for (int e = 0; e < P; ++e) acc[c][e] = cfma_conj(acc[c][e], rt[e], vv[e]);  // + vv conj(rt), 4 FMAs
      }
    } else {
      float2 rt[P];
      const float2* tc = p.twC + f1 * L;
#pragma unroll
      for (int e = 0; e < P; ++e) rt[e] = ldu(tc, (uint32_t)(t + T * e));
      if (chunk != 0) {
        const float2 u = unit_root_R<L, R>(p.twN, f1 * chunk);
#pragma unroll
        for (int e = 0; e < P; ++e) rt[e] = cmul(rt[e], u);
      }
#pragma unroll
      for (int e = 0; e < P; ++e) acc[0][e] = cfma_conj(acc[0][e], rt[e], vv[e]);
    }
  };
  // (prefetching the next class into a second register set measured slower
  // than register-resident twiddles, which need those registers)
#pragma unroll 1
  for (int f1 = f1_0; f1 < f1_1; ++f1) {
    float2 va[P], ha[P];
    load(va, ha, f1);
    prod(va, ha);
    step(va, f1);
  }
  float2* out = p.Pws + pg * p.p_stride + p.item_out[item];
  const float sc = 1.0f / (float)(L * R);
  if constexpr (C > 0) {
#pragma unroll
    for (int c = 0; c < C; ++c)
#pragma unroll
      for (int e = 0; e < P; ++e) {
        const int d = c * L + t + T * e;
        if (d < Sc) out[d] = cscale(acc[c][e], sc);
      }
  } else {
    const float* wc = p.wc + p.w_base[k] + c0;
#pragma unroll
    for (int e = 0; e < P; ++e) {
      const int d = t + T * e;
      if (d < Sc) out[d] = cscale(acc[0][e], wc[d] * sc);
    }
  }
}

// x[n] = sum over the items covering n of their stored products; the items
// that can cover a sample are listed per tile of 256 samples.
template <int L, int R, bool SPLIT>
__global__ __launch_bounds__(256) void k_ola1d(Large1D p, float* __restrict__ x, int64_t batch, int G) {
  constexpr int N = L * R, TILES = N / 256;
  // one workgroup per (pair, tile): the tile's item list is uniform
  const int64_t pair = blockIdx.x / TILES;
  const int tile = (int)(blockIdx.x % TILES);
  const int n = tile * 256 + (int)threadIdx.x;
  const float2* base = p.Pws + pair * (SPLIT ? G : 1) * p.p_stride;
  float2 acc = make_float2(0.f, 0.f);
  const int j0 = p.tile_off[tile], j1 = p.tile_off[tile + 1];
  for (int j = j0; j < j1; ++j) {
    const int it = p.tile_items[j];
    int dd = n - p.item_oc[it];
    if (dd < 0) dd += N;
    if (dd < p.item_len[it]) {
      const float2* s = base + p.item_out[it] + dd;
      acc = cadd(acc, s[0]);
      if constexpr (SPLIT) {
#pragma unroll 4
        for (int g = 1; g < G; ++g) acc = cadd(acc, s[g * p.p_stride]);
      }
    }
  }
  const int64_t sa = 2 * pair, sb = sa + 1;
  x[sa * N + n] = acc.x;
  if (sb < batch) x[sb * N + n] = acc.y;
}

// (L, R, P) instantiations of the four-step kernels; P (points per thread)
// is a plan-time choice.
#define PC_FOR_EACH_LRP(X)                                                          \
  X(8192, 2, 16) X(8192, 4, 16) X(8192, 8, 16) X(8192, 16, 16)                     \
  X(6144, 2, 12) X(6144, 4, 12) X(6144, 8, 12) X(6144, 16, 12)                     \
  X(4096, 2, 16) X(4096, 4, 16) X(4096, 8, 16) X(4096, 16, 16)

bool fourstep_variant_supported(int L, int R, int P) {
#define PC_CASE(LL, RR, PP) \
  if (L == LL && R == RR && P == PP) return true;
  PC_FOR_EACH_LRP(PC_CASE)
#undef PC_CASE
  return false;
}

// Workgroups that the four-step kernels keep resident (two of 256 threads
// per compute unit at their 237 to 256 VGPRs, one of 512): with fewer, the
// terms, classes or pairs are split further.  Measured (5 signals of 24576
// samples, 9 terms; us per launch at 24 points per thread and one group,
// split, and split at 12 points): forward 119, 25, 13.4; adjoint 60, 21,
// 11.9; gradient 60, 29, 11.3 (12 to 36 workgroups before, 108 split).  Fewer
// leave units idle, more run a second round (us per forward and adjoint at a
// target of 128, 256, 512 and 1024: 5 signals of 65536, 17 terms 44 and 50, 32
// and 40, 36 and 37, 58 and 49; 9 of them 65 and 73, 41 and 52, 38 and 42, 49
// and 49; 5 of 49152, one of 512 threads resident, 31 and 41, 28 and 35, 39
// and 40, 39 and 40).
static int64_t large_target(const Large1D& p) { return p.L / p.P >= 512 ? 256 : 512; }

int fwd1d_large_groups(const Large1D& p, int64_t pairs) {
  const int g = (int)std::min<int64_t>(p.m, std::max<int64_t>(1, large_target(p) / (pairs * p.R)));
  const int per = (p.m + g - 1) / g;  // terms per group; the fewest groups with that many
  return (p.m + per - 1) / per;
}

int adj1d_large_groups(const Large1D& p, int64_t pairs) {
  int g = 1;
  while (g < p.R && pairs * std::max(p.n_items, 1) * g * 2 <= large_target(p)) g *= 2;
  return g;
}

int grad1d_large_groups(const Large1D& p, int64_t pairs) {
  return (int)std::min<int64_t>(pairs, std::max<int64_t>(1, large_target(p) / ((int64_t)p.m * p.R)));
}

template <int L, int R, int P>
static LaunchStatus fold_fft_t(const Large1D& p, const float* x, int64_t n_sig, float2* out, bool pairs,
                               hipStream_t s, Tracer* tr) {
  const int64_t nb = pairs ? (n_sig + 1) / 2 : n_sig;
  TraceScope ts(tr, "fold_fft", s);
  hipLaunchKernelGGL((k_fold_fft<L, R, P>), dim3((unsigned)(nb * R)), dim3(L / P), 0, s, x, n_sig, pairs, out, p.tw,
                     p.twC, p.twN, p.zeros);
  return hipGetLastError();
}

#define PC_SPLIT_LAUNCH(K, C, ...)                                              \
  do {                                                                          \
    if (G > 1)                                                                  \
      hipLaunchKernelGGL((K<L, R, P, C, true>), grid, block, 0, s, __VA_ARGS__);  \
    else                                                                        \
      hipLaunchKernelGGL((K<L, R, P, C, false>), grid, block, 0, s, __VA_ARGS__); \
  } while (0)

template <int L, int R, int P>
static LaunchStatus fwd1d_large_t(const Large1D& p, const float* u, float* y, int64_t batch, hipStream_t s,
                                  Tracer* tr) {
  const int64_t pairs = (batch + 1) / 2;
  const int G = fwd1d_large_groups(p, pairs);
  {
    TraceScope ts(tr, "fwd1d_large", s);
    const dim3 grid((unsigned)(pairs * R * G)), block(L / P);
    if (p.chunks == 2)
      PC_SPLIT_LAUNCH(k_fwd1d_large, 2, u, batch, p, G);
    else if (p.chunks == 1)
      PC_SPLIT_LAUNCH(k_fwd1d_large, 1, u, batch, p, G);
    else
      PC_SPLIT_LAUNCH(k_fwd1d_large, 0, u, batch, p, G);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  // few pairs: smaller workgroups, so that every compute unit gets one
  const int64_t nthr = pairs * (L / 2);
  const unsigned nt = nthr < 256 * 256 ? 64 : 256;
  const dim3 grid((unsigned)((nthr + nt - 1) / nt)), block(nt);
  TraceScope ts(tr, "combine1d", s);
  if (G > 1)
    hipLaunchKernelGGL((k_combine1d<L, R, P, true>), grid, block, 0, s, p.Bws, y, batch, p.twC, G);
  else
    hipLaunchKernelGGL((k_combine1d<L, R, P, false>), grid, block, 0, s, p.Bws, y, batch, p.twC, G);
  return hipGetLastError();
}

template <int L, int R, int P>
static LaunchStatus adj1d_large_t(const Large1D& p, const float* v, float* x, int64_t batch, hipStream_t s,
                                  Tracer* tr) {
  const int64_t pairs = (batch + 1) / 2;
  LaunchStatus e = v ? fold_fft_t<L, R, P>(p, v, batch, p.Vws, true, s, tr) : hipSuccess;
  if (e != hipSuccess) return e;
  const int G = adj1d_large_groups(p, pairs);
  if (p.n_items > 0) {
    TraceScope ts(tr, "adj1d_large", s);
    const dim3 grid((unsigned)(pairs * p.n_items * G)), block(L / P);
    if (p.chunks == 2)
      PC_SPLIT_LAUNCH(k_adj1d_large, 2, p, G);
    else if (p.chunks == 1)
      PC_SPLIT_LAUNCH(k_adj1d_large, 1, p, G);
    else
      PC_SPLIT_LAUNCH(k_adj1d_large, 0, p, G);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  TraceScope ts(tr, "ola1d", s);
  const dim3 grid((unsigned)(pairs * (L * R / 256))), block(256);
  if (G > 1)
    hipLaunchKernelGGL((k_ola1d<L, R, true>), grid, block, 0, s, p, x, batch, G);
  else
    hipLaunchKernelGGL((k_ola1d<L, R, false>), grid, block, 0, s, p, x, batch, G);
  return hipGetLastError();
}

LaunchStatus launch_fold_fft(const Large1D& p, const float* x, int64_t n_sig, float2* out, bool pairs,
                             hipStream_t s, Tracer* tr) {
#define PC_CASE(LL, RR, PP) \
  if (p.L == LL && p.R == RR && p.P == PP) return fold_fft_t<LL, RR, PP>(p, x, n_sig, out, pairs, s, tr);
  PC_FOR_EACH_LRP(PC_CASE)
#undef PC_CASE
  return hipErrorInvalidValue;
}

LaunchStatus launch_fwd1d_large(const Large1D& p, const float* u, float* y, int64_t batch, hipStream_t s,
                                Tracer* tr) {
#define PC_CASE(LL, RR, PP) \
  if (p.L == LL && p.R == RR && p.P == PP) return fwd1d_large_t<LL, RR, PP>(p, u, y, batch, s, tr);
  PC_FOR_EACH_LRP(PC_CASE)
#undef PC_CASE
  return hipErrorInvalidValue;
}

LaunchStatus launch_adj1d_large(const Large1D& p, const float* v, float* x, int64_t batch, hipStream_t s,
                                Tracer* tr) {
#define PC_CASE(LL, RR, PP) \
  if (p.L == LL && p.R == RR && p.P == PP) return adj1d_large_t<LL, RR, PP>(p, v, x, batch, s, tr);
  PC_FOR_EACH_LRP(PC_CASE)
#undef PC_CASE
  return hipErrorInvalidValue;
}

// ===========================================================================
// Spectra as parameters: import / export in the natural half-spectrum layout
// spec[k][f], f <= N/2 (the layout of a real FFT), and the gradient of a
// scalar loss with respect to them.
//
// The internal spectra are full and Hermitian (they multiply pair-packed
// complex signals), so an imported half-spectrum is extended by conjugate
// symmetry with the imaginary parts at DC and Nyquist dropped, the values an
// inverse real transform ignores.
//
// Gradient: with Z = F^*(w_k . u) and Gh = F^*(dL/dy) for a real signal, the
// gradient with respect to spec[k][f] (convention dL/dRe + i dL/dIm) is
// (c_f / N) conj(Z[f]) Gh[f], c_f = 1 at DC and Nyquist, 2 elsewhere.  For a
// pair-packed signal with full spectra A = F^*(w_k . (u_a + i u_b)) and
// C = F^*(g_a + i g_b), the sum over the two signals of conj(Z[f]) Gh[f] is
// (E[f] + conj(E[-f])) / 2 with E = conj(A) . C, so the kernels accumulate E
// over pairs and combine f with -f at the end.
// ===========================================================================

__device__ __forceinline__ float half_weight(int f, int n) { return (f == 0 || 2 * f == n) ? 1.f : 2.f; }

__device__ __forceinline__ float2 hermitian_value(const float2* __restrict__ half, int f, int n) {
  if (2 * f <= n) {
    float2 v = half[f];
    if (f == 0 || 2 * f == n) v.y = 0.f;
    return v;
  }
  return cconj(half[n - f]);
}

template <int L>
__global__ __launch_bounds__(256) void k_import1d_small(const float2* __restrict__ spec, float2* __restrict__ H, int m) {
  const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= (int64_t)m * L) return;
  const int k = (int)(gid / L), f = (int)(gid % L);
  H[gid] = hermitian_value(spec + (int64_t)k * (L / 2 + 1), f, L);
}

template <int L>
__global__ __launch_bounds__(256) void k_export1d_small(const float2* __restrict__ H, float2* __restrict__ spec,
                                                        int m) {
  constexpr int NH = L / 2 + 1;
  const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= (int64_t)m * NH) return;
  const int k = (int)(gid / NH), f = (int)(gid % NH);
  spec[gid] = H[(int64_t)k * L + f];
}

// Full spectra of pair-packed signals: out[pair][f] = F^*(x_a + i x_b)[f].
template <int L>
__global__ __launch_bounds__(ffts_per_block(L) * fft_threads(L)) void k_fft_pairs_small(
    const float* __restrict__ x, int64_t batch, float2* __restrict__ out, const float2* __restrict__ tw) {
  constexpr int P = points_per_thread(L), T = L / P, NF = ffts_per_block(L);
  __shared__ float2 lds[NF * lds_len<L>()];
  __shared__ float2 twl[L];
  stage_twiddles<L>(twl, tw);
  const int c = threadIdx.x / T, t = threadIdx.x % T;
  const int64_t pair = (int64_t)blockIdx.x * NF + c;
  const int64_t sa = 2 * pair, sb = sa + 1;
  const bool va = sa < batch, vb = sb < batch;
  float2 v[P];
#pragma unroll
  for (int e = 0; e < P; ++e) {
    const int n = t + T * e;
    v[e] = make_float2(va ? x[sa * L + n] : 0.f, vb ? x[sb * L + n] : 0.f);
  }
  fft_wg<L, P, false>(v, lds + c * lds_len<L>(), twl, t);
  if (va) {
#pragma unroll
    for (int e = 0; e < P; ++e) out[pair * L + t + T * e] = v[e];
  }
}

// (512 threads up to 1024 points: more terms per workgroup)
constexpr int split_slots(int L) { return split_threads(L) >= 256 ? 1 : (L <= 1024 ? 512 : 256) / split_threads(L); }

// Backward of the small sizes.  Slot c of workgroup (kg, pg) owns term
// k = kg NF + c and takes pairs pg, pg + PG, ...: from one transform of the
// pair's output gradient, V, it accumulates E_k += conj(F^*(w_k u)) . V over
// its pairs and, with GU, forms w_k . F(conj(H_k) V), whose sum over the
// workgroup's slots is the workgroup's share of dL/du.  k_bwd1d_small_sum
// adds the shares (dL/du over kg, E over pg) and writes both results.  The
// transform of the gradient is done again by every term group: these sizes
// are bound by latency, and a launch for it costs more; PRE reads it from Gc
// (k_fft_pairs_small), for term counts that fill the chip by themselves.
// Measured (both gradients, us; the pairs one after another in one workgroup
// per term group and a separate adjoint -> here): 16 signals of 3072 samples,
// 12 terms, 158 -> 16.5; 64 of 8192, 16 terms, 378 -> 48; 1 of 1024, 8 terms,
// 20.4 -> 14.6.
template <int L, bool GU, bool PRE>
__global__ __launch_bounds__(split_slots(L) * split_threads(L)) void k_bwd1d_small(
    const float* __restrict__ u, const float* __restrict__ gy, int64_t pairs, int64_t batch, int m,
    const float* __restrict__ w, const float2* __restrict__ H, const float2* __restrict__ tw, int KG, int PG,
    const float2* __restrict__ Gc, float2* __restrict__ gu_part, float2* __restrict__ e_part) {
  constexpr int P = split_points(L), T = L / P, NF = split_slots(L), NT = NF * T;
  __shared__ float2 lds[NF * lds_len<L>()];
  __shared__ float2 twl[L];
  const int tid = (int)threadIdx.x, c = tid / T, t = tid % T;
  const int kg = (int)(blockIdx.x % KG), pg = (int)(blockIdx.x / KG);
  TwStage<L, NT> ts;
  ts.load(tw, tid);
  const int kraw = kg * NF + c, k = kraw < m ? kraw : m - 1;
  const float live = kraw < m ? 1.f : 0.f;  // a slot past the last term adds nothing to dL/du
  const float* wk = w + (int64_t)k * L;
  float wv[P];
  float2 hv[GU ? P : 1];
#pragma unroll
  for (int e = 0; e < P; ++e) wv[e] = wk[t + T * e];
  if constexpr (GU) {
#pragma unroll
    for (int e = 0; e < P; ++e) hv[e] = H[(int64_t)k * L + t + T * e];
  }
  float2 acc[P];
#pragma unroll
  for (int e = 0; e < P; ++e) acc[e] = make_float2(0.f, 0.f);
  float2* my = lds + c * lds_len<L>();
  ts.commit(twl, tid);
  for (int64_t pr = pg; pr < pairs; pr += PG) {
    const bool vb = 2 * pr + 1 < batch;
    const int64_t o = 2 * pr * L, ob = vb ? L : 0;  // an odd batch's last pair: the signal again, zeroed
    float2 z[P], V[P];
#pragma unroll
    for (int e = 0; e < P; ++e) z[e] = make_float2(u[o + t + T * e], u[o + ob + t + T * e]);
#pragma unroll
    for (int e = 0; e < P; ++e)
      V[e] = PRE ? Gc[pr * L + t + T * e] : make_float2(gy[o + t + T * e], gy[o + ob + t + T * e]);
#pragma unroll
    for (int e = 0; e < P; ++e) {
      z[e] = make_float2(wv[e] * z[e].x, vb ? wv[e] * z[e].y : 0.f);
      if (!PRE && !vb) V[e].y = 0.f;
    }
    if constexpr (!PRE) fft_wv<L, P, false, SYNC_WAVE>(V, my, twl, opaque1d(t));
    fft_wv<L, P, false, SYNC_WAVE>(z, my, twl, opaque1d(t));
#pragma unroll
    for (int e = 0; e < P; ++e) acc[e] = cfma_conj(acc[e], z[e], V[e]);
    if constexpr (GU) {
#pragma unroll
      for (int e = 0; e < P; ++e) V[e] = cmulc(V[e], hv[e]);
      fft_wv<L, P, true, SYNC_WAVE>(V, my, twl, opaque1d(t));
      float2* mine = gu_part + (pr * KG + kg) * L;
      if constexpr (NF == 1) {
#pragma unroll
        for (int e = 0; e < P; ++e) mine[t + T * e] = cscale(V[e], wv[e]);
      } else {
        __syncthreads();  // every slot is done with its exchange region
#pragma unroll
        for (int e = 0; e < P; ++e) lds[c * L + t + T * e] = cscale(V[e], live * wv[e]);
        __syncthreads();
        for (int n = tid; n < L; n += NT) {
          float2 a = lds[n];
#pragma unroll
          for (int q = 1; q < NF; ++q) a = cadd(a, lds[q * L + n]);
          mine[n] = a;
        }
        __syncthreads();  // the sums are read before the next pair's exchanges
      }
    }
  }
  if (kraw < m) {
    float2* ek = e_part + ((int64_t)k * PG + pg) * L;
#pragma unroll
    for (int e = 0; e < P; ++e) ek[t + T * e] = acc[e];
  }
}

// The sums of k_bwd1d_small's shares: blocks below gu_blocks write dL/du
// (scaled, both signals of a pair), the rest the spectra gradient
// gspec[k][f], f <= N/2, from E[f] and E[-f].
template <int L>
__global__ __launch_bounds__(256) void k_bwd1d_small_sum(const float2* __restrict__ gu_part,
                                                         const float2* __restrict__ e_part, int KG, int PG, int m,
                                                         int64_t batch, unsigned gu_blocks, float* __restrict__ gu,
                                                         float2* __restrict__ gspec) {
  constexpr int NH = L / 2 + 1;
  const float sc = 1.0f / (float)L;
  if (blockIdx.x < gu_blocks) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t pair = i / L;
    const int n = (int)(i % L);
    if (2 * pair >= batch) return;
    const float2* s = gu_part + pair * KG * L + n;
    float2 a = s[0];
#pragma unroll 8
    for (int g = 1; g < KG; ++g) a = cadd(a, s[(int64_t)g * L]);
    gu[2 * pair * L + n] = a.x * sc;
    if (2 * pair + 1 < batch) gu[(2 * pair + 1) * L + n] = a.y * sc;
    return;
  }
  const int64_t i = (int64_t)(blockIdx.x - gu_blocks) * 256 + threadIdx.x;
  if (i >= (int64_t)m * NH) return;
  const int k = (int)(i / NH), f = (int)(i % NH), fm = f == 0 ? 0 : L - f;
  const float2* e = e_part + (int64_t)k * PG * L;
  float2 a = e[f], b = e[fm];
#pragma unroll 4
  for (int g = 1; g < PG; ++g) {
    a = cadd(a, e[(int64_t)g * L + f]);
    b = cadd(b, e[(int64_t)g * L + fm]);
  }
  const float s = 0.5f * half_weight(f, L) / (float)L;
  gspec[i] = make_float2(s * (a.x + b.x), s * (a.y - b.y));
}

// ---- four-step layout -------------------------------------------------------

// The four-step path stores its spectra in the frame of each window's origin
// o_k: Hd[k][f1][f2] = H_k[f] W_N^{f o_k}, f = f1 + R f2.
template <int L, int R>
__device__ __forceinline__ float2 origin_phase(const float2* __restrict__ twN, int f, int o) {
  constexpr int N = L * R;
  return twN[(int)(((int64_t)f * o) % N)];
}

template <int L, int R, int P>
__global__ __launch_bounds__(256) void k_import1d_large(const float2* __restrict__ spec, float2* __restrict__ Hd,
                                                        int m, const int* __restrict__ w_off,
                                                        const float2* __restrict__ twN) {
  constexpr int N = L * R;
  const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= (int64_t)m * N) return;
  const int k = (int)(gid / N);
  const int rem = (int)(gid % N);
  const int f = rem / L + R * block_elem<L, P>(rem % L);
  Hd[gid] = cmul(hermitian_value(spec + (int64_t)k * (N / 2 + 1), f, N), origin_phase<L, R>(twN, f, w_off[k]));
}

template <int L, int R, int P>
__global__ __launch_bounds__(256) void k_export1d_large(const float2* __restrict__ Hd, float2* __restrict__ spec,
                                                        int m, const int* __restrict__ w_off,
                                                        const float2* __restrict__ twN) {
  constexpr int N = L * R, NH = N / 2 + 1;
  const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= (int64_t)m * NH) return;
  const int k = (int)(gid / NH), f = (int)(gid % NH);
  spec[gid] =
      cmulc(Hd[((int64_t)k * R + f % R) * L + block_pos(f / R, L / P)], origin_phase<L, R>(twN, f, w_off[k]));
}

// In place: natural-frame spectra (from the whole-signal transform of h_k)
// to the window-origin frame.
template <int L, int R, int P>
__global__ __launch_bounds__(256) void k_origin_phase1d(float2* __restrict__ Hd, int m, const int* __restrict__ w_off,
                                                        const float2* __restrict__ twN) {
  constexpr int N = L * R;
  const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= (int64_t)m * N) return;
  const int k = (int)(gid / N);
  const int rem = (int)(gid % N);
  const int f = rem / L + R * block_elem<L, P>(rem % L);
  Hd[gid] = cmul(Hd[gid], origin_phase<L, R>(twN, f, w_off[k]));
}

// E_k^{f1} = sum over pairs of conj(FFT_L(fold(w_k u))) . Gdec^{f1}, one
// (term, class, pair group) per workgroup: group g of G takes pairs g, g + G,
// ... and writes slice g of E (k_grad_export1d_large adds the slices).
template <int L, int R, int P, int C>
__global__ __launch_bounds__(L / P) void k_grad1d_large(const float* __restrict__ u, int64_t batch, Large1D p,
                                                        float2* __restrict__ E, int G) {
  constexpr int N = L * R;
  __shared__ float2 lds[fs_lds_len<L, P>()];
  FsLds<L, P> xl(lds);
  const int t = threadIdx.x;
  float2 twr[tw_reg_count<L, P>()];
  load_tw_reg<L, P>(twr, p.tw, t);
  const int f1 = blockIdx.x % R;
  const int k = (blockIdx.x / R) % p.m, g = blockIdx.x / R / p.m;
  const int S = p.w_len[k];
  const int o = p.w_off[k];
  const float* wc = p.wc + p.w_base[k];
  (void)wc;
  float2 acc[P];
#pragma unroll
  for (int e = 0; e < P; ++e) acc[e] = make_float2(0.f, 0.f);
  const int64_t pairs = (batch + 1) / 2;
  if (S > 0) {
    for (int64_t pr = g; pr < pairs; pr += G) {
      const float* xa = u + 2 * pr * N;
      const float* xb = 2 * pr + 1 < batch ? xa + N : p.zeros;
      // an opaque index: the compiler otherwise keeps the window table's
      // values (the same for every pair) and the addresses in registers for
      // the whole loop (362 registers at 4096 points, 384 bytes of spills at
      // 6144); the gradient's spectrum is read after the transform, which
      // leaves more waves
      const int tt = opaque1d(t);
      float2 v[P];
      if constexpr (C > 0)
        fold_short<L, R, P, C>(v, tt, xa, xb, o, p.cw + ((int64_t)k * R + f1) * C * L);
      else
        fold_long<L, R, P>(v, tt, f1, xa, xb, wc, o, S, p.twC, p.twN);
      xl.template fft<false>(v, twr, t);
      float2 gv[P];
      load_blk<L, P>(p.Vws + (pr * R + f1) * L, gv, tt);
#pragma unroll
      for (int e = 0; e < P; ++e) acc[e] = cfma_conj(acc[e], v[e], gv[e]);
    }
  }
  store_blk<L, P>(E + (((int64_t)g * p.m + k) * R + f1) * L, acc, t);
}

template <int L, int R, int P>
__global__ __launch_bounds__(256) void k_grad_export1d_large(const float2* __restrict__ E, float2* __restrict__ gspec,
                                                             int m, const int* __restrict__ w_off,
                                                             const float2* __restrict__ twN, int G) {
  constexpr int N = L * R, NH = N / 2 + 1;
  const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= (int64_t)m * NH) return;
  const int k = (int)(gid / NH), f = (int)(gid % NH);
  const int fm = (N - f) % N;
  // E was accumulated with the windowed transforms in the window-origin
  // frame; the natural-frame product carries conj(W_N^{f o_k})
  constexpr int T = L / P;
  const float2* ea = E + ((int64_t)k * R + f % R) * L + block_pos(f / R, T);
  const float2* eb = E + ((int64_t)k * R + fm % R) * L + block_pos(fm / R, T);
  float2 sa = ea[0], sb = eb[0];
#pragma unroll 4
  for (int g = 1; g < G; ++g) {
    sa = cadd(sa, ea[(int64_t)g * m * N]);
    sb = cadd(sb, eb[(int64_t)g * m * N]);
  }
  const float2 a = cmulc(sa, origin_phase<L, R>(twN, f, w_off[k]));
  const float2 b = cmulc(sb, origin_phase<L, R>(twN, fm, w_off[k]));
  const float sc = 0.5f * half_weight(f, N) / (float)N;
  gspec[gid] = make_float2(sc * (a.x + b.x), sc * (a.y - b.y));
}

// out[i] = conj(in[i]); in may equal out
__global__ __launch_bounds__(256) void k_conj(const float2* in, float2* out, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = cconj(in[i]);
}

// ---- launchers --------------------------------------------------------------

static inline unsigned blocks_for(int64_t n) { return (unsigned)((n + 255) / 256); }

LaunchStatus launch_conj(const float2* in, float2* out, int64_t n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_conj, dim3(blocks_for(n)), dim3(256), 0, s, in, out, n);
  return hipGetLastError();
}

LaunchStatus launch_spectra1d(const Small1D* ps, const Large1D* pl, const float2* in, float2* out, bool import,
                              hipStream_t s) {
  if (ps) {
    const Small1D& p = *ps;
    switch (p.L) {
#define PC_CASE(LL)                                                                                              \
  case LL:                                                                                                       \
    if (import)                                                                                                  \
      hipLaunchKernelGGL(k_import1d_small<LL>, dim3(blocks_for((int64_t)p.m * LL)), dim3(256), 0, s, in,         \
                         const_cast<float2*>(p.H), p.m);                                                         \
    else                                                                                                         \
      hipLaunchKernelGGL(k_export1d_small<LL>, dim3(blocks_for((int64_t)p.m * (LL / 2 + 1))), dim3(256), 0, s,   \
                         p.H, out, p.m);                                                                         \
    return hipGetLastError();
      PC_FOR_EACH_L(PC_CASE)
#undef PC_CASE
    }
    return hipErrorInvalidValue;
  }
  const Large1D& p = *pl;
#define PC_CASE(LL, RR, PP)                                                                                     \
  if (p.L == LL && p.R == RR && p.P == PP) {                                                                    \
    if (import)                                                                                                 \
      hipLaunchKernelGGL((k_import1d_large<LL, RR, PP>), dim3(blocks_for((int64_t)p.m * LL * RR)), dim3(256), 0, \
                         s, in, const_cast<float2*>(p.Hd), p.m, p.w_off, p.twN);                                \
    else                                                                                                        \
      hipLaunchKernelGGL((k_export1d_large<LL, RR, PP>), dim3(blocks_for((int64_t)p.m * (LL * RR / 2 + 1))),    \
                         dim3(256), 0, s, p.Hd, out, p.m, p.w_off, p.twN);                                      \
    return hipGetLastError();                                                                                   \
  }
  PC_FOR_EACH_LRP(PC_CASE)
#undef PC_CASE
  return hipErrorInvalidValue;
}

LaunchStatus launch_origin_phase1d(const Large1D& p, float2* Hd, hipStream_t s) {
#define PC_CASE(LL, RR, PP)                                                                                  \
  if (p.L == LL && p.R == RR && p.P == PP) {                                                                 \
    hipLaunchKernelGGL((k_origin_phase1d<LL, RR, PP>), dim3(blocks_for((int64_t)p.m * LL * RR)), dim3(256), 0, \
                       s, Hd, p.m, p.w_off, p.twN);                                                          \
    return hipGetLastError();                                                                                \
  }
  PC_FOR_EACH_LRP(PC_CASE)
#undef PC_CASE
  return hipErrorInvalidValue;
}

// Term groups (one term per slot) and pair groups (about one workgroup per
// compute unit) of a small backward; PRE (see the kernel) from 256 term
// groups on, where the second transform per term and pair would cost
// throughput.
struct Bwd1D {
  int KG, PG;
  bool pre, gu;  // gu: dL/du fits (shares of at most 64 MB)
};
template <int L>
static Bwd1D bwd1d_t(int m, int64_t pairs) {
  constexpr int SF = split_slots(L);
  Bwd1D q;
  q.KG = (m + SF - 1) / SF;
  q.PG = (int)std::min<int64_t>(pairs, std::max<int64_t>(1, 256 / q.KG));
  q.pre = q.KG >= 256;
  q.gu = !q.pre && pairs * q.KG * L <= ((int64_t)1 << 23);
  return q;
}

template <int L>
static int64_t bwd1d_small_work_t(int m, int64_t pairs) {
  const Bwd1D q = bwd1d_t<L>(m, pairs);
  return ((int64_t)m * q.PG + (q.pre ? pairs : q.gu ? pairs * q.KG : 0)) * L;
}

int64_t bwd1d_small_work(int L, int m, int64_t pairs) {
  switch (L) {
#define PC_CASE(LL) \
  case LL:          \
    return bwd1d_small_work_t<LL>(m, pairs);
    PC_FOR_EACH_L(PC_CASE)
#undef PC_CASE
  }
  return 0;
}

bool bwd1d_small_gu(int L, int m, int64_t pairs) {
  switch (L) {
#define PC_CASE(LL) \
  case LL:          \
    return bwd1d_t<LL>(m, pairs).gu;
    PC_FOR_EACH_L(PC_CASE)
#undef PC_CASE
  }
  return false;
}

template <int L>
static LaunchStatus bwd1d_small_t(const Small1D& p, const float* u, const float* gy, float* gu, float2* gspec,
                                  int64_t batch, float2* work, hipStream_t s) {
  const int64_t pairs = (batch + 1) / 2;
  const Bwd1D q = bwd1d_t<L>(p.m, pairs);
  if (gu && !q.gu) return hipErrorInvalidValue;
  float2* rest = work + (int64_t)p.m * q.PG * L;  // the shares of dL/du, or Gc
  const dim3 grid((unsigned)(q.KG * q.PG)), block(split_slots(L) * split_threads(L));
  if (q.pre) {
    constexpr int NF = ffts_per_block(L), T = fft_threads(L);
    hipLaunchKernelGGL(k_fft_pairs_small<L>, dim3((unsigned)((pairs + NF - 1) / NF)), dim3(NF * T), 0, s, gy, batch,
                       rest, p.tw);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_bwd1d_small<L, false, true>), grid, block, 0, s, u, gy, pairs, batch, p.m, p.w, p.H, p.tws,
                       q.KG, q.PG, rest, rest, work);
  } else if (gu) {
    hipLaunchKernelGGL((k_bwd1d_small<L, true, false>), grid, block, 0, s, u, gy, pairs, batch, p.m, p.w, p.H, p.tws,
                       q.KG, q.PG, nullptr, rest, work);
  } else {
    hipLaunchKernelGGL((k_bwd1d_small<L, false, false>), grid, block, 0, s, u, gy, pairs, batch, p.m, p.w, p.H, p.tws,
                       q.KG, q.PG, nullptr, rest, work);
  }
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const unsigned gub = gu ? blocks_for(pairs * L) : 0;
  hipLaunchKernelGGL(k_bwd1d_small_sum<L>, dim3(gub + blocks_for((int64_t)p.m * (L / 2 + 1))), dim3(256), 0, s, rest,
                     work, q.KG, q.PG, p.m, batch, gub, gu, gspec);
  return hipGetLastError();
}

LaunchStatus launch_bwd1d_small(const Small1D& p, const float* u, const float* gy, float* gu, float2* gspec,
                                int64_t batch, float2* work, hipStream_t s, Tracer* tr) {
  TraceScope ts(tr, gu ? "bwd1d_small" : "grad1d_small", s);
  switch (p.L) {
#define PC_CASE(LL) \
  case LL:          \
    return bwd1d_small_t<LL>(p, u, gy, gu, gspec, batch, work, s);
    PC_FOR_EACH_L(PC_CASE)
#undef PC_CASE
  }
  return hipErrorInvalidValue;
}

template <int L, int R, int P>
static LaunchStatus grad1d_large_t(const Large1D& p, const float* u, const float* gy, float2* gspec, int64_t batch,
                                   float2* E, hipStream_t s, Tracer* tr) {
  LaunchStatus e = fold_fft_t<L, R, P>(p, gy, batch, p.Vws, true, s, tr);
  if (e != hipSuccess) return e;
  const int G = grad1d_large_groups(p, (batch + 1) / 2);
  {
    TraceScope ts(tr, "grad1d_large", s);
    const dim3 grid((unsigned)(p.m * R * G)), block(L / P);
    if (p.chunks == 2)
      hipLaunchKernelGGL((k_grad1d_large<L, R, P, 2>), grid, block, 0, s, u, batch, p, E, G);
    else if (p.chunks == 1)
      hipLaunchKernelGGL((k_grad1d_large<L, R, P, 1>), grid, block, 0, s, u, batch, p, E, G);
    else
      hipLaunchKernelGGL((k_grad1d_large<L, R, P, 0>), grid, block, 0, s, u, batch, p, E, G);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL((k_grad_export1d_large<L, R, P>), dim3(blocks_for((int64_t)p.m * (L * R / 2 + 1))), dim3(256), 0,
                     s, E, gspec, p.m, p.w_off, p.twN, G);
  return hipGetLastError();
}

LaunchStatus launch_grad1d_large(const Large1D& p, const float* u, const float* gy, float2* gspec, int64_t batch,
                                 float2* E, hipStream_t s, Tracer* tr) {
#define PC_CASE(LL, RR, PP) \
  if (p.L == LL && p.R == RR && p.P == PP) return grad1d_large_t<LL, RR, PP>(p, u, gy, gspec, batch, E, s, tr);
  PC_FOR_EACH_LRP(PC_CASE)
#undef PC_CASE
  return hipErrorInvalidValue;
}

}  // namespace pc
