// Which samples of its rows the projection's contraction reads (k_gemm_nt_f32
// in kern_construct.hip): constants and arithmetic shared by the kernel, the
// host's launch and the CPU test that walks every chunk of a call.
#pragma once
#include <cstdint>

namespace pc {

constexpr int GEMM_ROWS = 64, GEMM_COLS = 32, GEMM_KT = 64, GEMM_CHUNK = 512;

// Stages of GEMM_KT samples per segment and segments of the contraction: about
// five workgroups per CU (enough that the last round costs little), as few
// segments as that needs.
constexpr int gemm_seg_stages(int64_t rows, int m, int64_t K) {
  const int64_t tiles =
      ((rows + GEMM_ROWS - 1) / GEMM_ROWS + (m + GEMM_ROWS - 1) / GEMM_ROWS) * ((m + GEMM_COLS - 1) / GEMM_COLS);
  const int64_t stages = (K + GEMM_KT - 1) / GEMM_KT, want = (1280 + tiles - 1) / tiles;
  const int64_t segs = stages < want ? stages : want;
  return (int)((stages + segs - 1) / segs);
}
constexpr int gemm_segments(int64_t rows, int m, int64_t K) {
  const int64_t per = gemm_seg_stages(rows, m, K), stages = (K + GEMM_KT - 1) / GEMM_KT;
  return (int)((stages + per - 1) / per);
}
// stages of a segment that has k_left samples from its first to the row's end
constexpr int gemm_stages(int64_t k_left, int seg_stages) {
  return (int)(k_left < (int64_t)seg_stages * GEMM_KT ? (k_left + GEMM_KT - 1) / GEMM_KT : seg_stages);
}

// Chunk c (4 samples) of a segment's stage s: whether it lies before the row's
// end, and the offset from the segment's first sample at which it is read.
// (K need not be whole stages: a chunk past the end reads the segment's first
// samples, which every segment has, and counts as zero.)
constexpr bool gemm_chunk_inside(int s, int c, int64_t k_left) { return (int64_t)s * GEMM_KT + 4 * c < k_left; }
constexpr int64_t gemm_chunk_offset(int s, int c, int64_t k_left) {
  return gemm_chunk_inside(s, c, k_left) ? (int64_t)s * GEMM_KT + 4 * c : 0;
}

}  // namespace pc
