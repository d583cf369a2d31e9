"""The projection's contraction stays inside its rows (no GPU needed): the
arithmetic the kernel reads by (csrc/project_tile.hpp) compiled for the host
and walked over every chunk of every stage that a workgroup loads."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1604_04374_amd", "csrc")

WALK = r"""
#include <cstdio>
#include <vector>
#include "project_tile.hpp"
using namespace pc;
int main() {
  long long calls = 0;
  for (int64_t K = 16; K <= 8192; K += 16)
    for (int m : {1, 16, 33, 128})
      for (int64_t rows : {(int64_t)1, (int64_t)65, (int64_t)1000, K}) {
        if (rows > K) continue;
        const int per = gemm_seg_stages(rows, m, K), segs = gemm_segments(rows, m, K);
        std::vector<int> used((size_t)K / 4, 0);
        for (int z = 0; z < segs; ++z) {
          const int64_t k0 = (int64_t)z * per * GEMM_KT, left = K - k0;
          const int ns = gemm_stages(left, per);
          // stages 0 to 2 are loaded ahead, then s + 3 behind every stage s
          for (int s = 0; s < ns + 3; ++s)
            for (int c = 0; c < GEMM_KT / 4; ++c) {
              const int64_t at = k0 + gemm_chunk_offset(s, c, left);
              if (at < 0 || at + 4 > K) {
                std::printf("n %lld m %d rows %lld segment %d stage %d chunk %d reads sample %lld\n", (long long)K, m,
                            (long long)rows, z, s, c, (long long)at);
                return 1;
              }
              if (!gemm_chunk_inside(s, c, left) || s >= ns) continue;
              if (at != k0 + (int64_t)s * GEMM_KT + 4 * c) return 2;
              ++used[(size_t)at / 4];
            }
        }
        for (int u : used)
          if (u != 1) return 3;  // every sample once
        ++calls;
      }
  std::printf("%lld calls\n", calls);
  return 0;
}
"""


def test_contraction_reads_inside_its_rows(tmp_path):
    src, exe = tmp_path / "walk.cpp", tmp_path / "walk"
    src.write_text(WALK)
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", CSRC, "-o", str(exe), str(src)], check=True, timeout=120)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout or f"exit {r.returncode}"
