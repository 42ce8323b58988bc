"""The choice of tile and split of the products (gemm_plan.h, host code): every
plan covers its product, leaves no split empty and stays inside the workspace
it was given, for any workspace and compute-unit count."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2405_14009_amd", "csrc")

MAIN = r"""
#include <cstdio>
#include "gemm_plan.h"
int main() {
  const long dims[] = {8, 24, 32, 40, 64, 136, 256, 264, 640, 1024, 1288, 3072, 5120, 16384};
  const long depths[] = {8, 64, 72, 512, 1000, 2048, 6000, 32768, 65536};
  const long rooms[] = {0, 4096, 1L << 20, 16L << 20};
  long n = 0, splits = 0;
  auto bad = [](const char* what, long M, long N, long K, long room, int cus) {
    std::printf("%s: M %ld N %ld K %ld room %ld cus %d\n", what, M, N, K, room, cus);
    return 1;
  };
  for (long M : dims) for (long N : dims) for (long K : depths) for (long room : rooms) for (int cus : {64, 256, 304}) {
    for (int tn = 0; tn < 2; ++tn) {
      // column sums: none, and the least room that a caller provides
      for (long cs : {-1L, (M + 255) / 256 * N}) {
        const GemmPlan p = plan_bf16(M, N, K, tn, 1, room, cs, cus);
        if (p.tiles != (M + p.bm - 1) / p.bm * ((N + p.bn - 1) / p.bn)) return bad("tiles", M, N, K, room, cus);
        if (p.split_k % 64 || p.splits * (long)p.split_k < K || (p.splits - 1) * (long)p.split_k >= K)
          return bad("bf16 splits", M, N, K, room, cus);
        if (p.split_floats > room || (p.splits > 1) != (p.split_floats > 0)) return bad("bf16 room", M, N, K, room, cus);
        if (cs >= 0 && p.colsum_rows(M) * N > cs) return bad("column sums", M, N, K, room, cus);
        if (tn && p.tile == TILE_192x256) return bad("192 rows", M, N, K, room, cus);
        ++n;
        splits += p.splits > 1;
      }
    }
    for (long nseg : {1L, 3L}) {
      const long k = nseg * ((K + 31) / 32 * 32);
      const F32Plan p = plan_f32(M, N, nseg, K, 1, room, cus);
      if (p.tiles != (M + p.bm - 1) / p.bm * ((N + p.bm - 1) / p.bm)) return bad("f32 tiles", M, N, K, room, cus);
      if (p.split_k % 32 || p.splits * (long)p.split_k < k || (p.splits - 1) * (long)p.split_k >= k)
        return bad("f32 splits", M, N, K, room, cus);
      if (p.split_floats > room) return bad("f32 room", M, N, K, room, cus);
    }
  }
  std::printf("%ld plans, %ld split\n", n, splits);
  return splits > 0 ? 0 : 1;
}
"""


def test_plans_cover_and_fit(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("no host compiler")
    src = tmp_path / "plan.cpp"
    src.write_text(MAIN)
    exe = tmp_path / "plan"
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
