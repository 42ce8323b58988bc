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


def compiled(tmp_path, main):
    if shutil.which("g++") is None:
        pytest.skip("no host compiler")
    src = tmp_path / "plan.cpp"
    src.write_text(main)
    exe = tmp_path / "plan"
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    return str(exe)


def test_plans_cover_and_fit(tmp_path):
    r = subprocess.run([compiled(tmp_path, MAIN)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout


# Unsplit products as timed alone on the card (us): weight-gradient layout or
# not, M, N, K, then 256x256, 256x128, 128x128, 64x64 and 192x256 tiles (0: not
# timed).  Partial rounds of large tiles, second rounds of tiles that share a
# compute unit, short and long reductions.
TIMED = [
    (0, 2048, 12288, 12288, (553, 508, 673, 0, 714)), (0, 2048, 12288, 36864, (1691, 1570, 0, 0, 2366)),
    (0, 2048, 36864, 12288, (1475, 1565, 0, 0, 1762)), (0, 2048, 20480, 5120, (377, 391, 485, 0, 424)),
    (0, 2048, 10240, 2048, (106, 100, 119, 186, 95)), (0, 4096, 1280, 5120, (118, 75, 92, 120, 105)),
    (0, 4096, 2048, 4096, (95, 63, 82, 151, 82)), (0, 4096, 3072, 4096, (97, 114, 157, 227, 145)),
    (0, 2048, 2560, 2560, (56, 36, 39, 59, 44)), (0, 512, 1024, 1024, (25, 18, 15, 8, 21)),
    (0, 2048, 4096, 16384, (355, 224, 314, 0, 316)),
    (1, 8192, 32768, 512, (652, 911, 719, 0, 0)), (1, 4096, 16384, 512, (143, 199, 164, 245, 0)),
    (1, 49152, 12288, 512, (1269, 1681, 1432, 0, 0)), (1, 1536, 6144, 4096, (107, 128, 116, 180, 0)),
    (1, 3072, 3072, 2048, (53, 75, 65, 96, 0)), (1, 1024, 4096, 4096, (84, 65, 53, 67, 0)),
    (1, 4096, 2560, 4096, (110, 129, 138, 209, 0)), (1, 12288, 12288, 2048, (643, 773, 860, 0, 0)),
]


def test_choice_on_timed_products(tmp_path):
    """Without split workspace the choice is within 6 % of the fastest tile."""
    exe = compiled(tmp_path, """
#include <cstdio>
#include "gemm_plan.h"
int main() {
  int tn;
  long M, N, K;
  while (std::scanf("%d %ld %ld %ld", &tn, &M, &N, &K) == 4) std::printf("%d\\n", (int)plan_bf16(M, N, K, tn, 1, 0, -1, 256).tile);
}
""")
    text = "".join("%d %d %d %d\n" % row[:4] for row in TIMED)
    out = subprocess.run([exe], input=text, capture_output=True, text=True, timeout=60, check=True).stdout.split()
    bad = []
    for row, tile in zip(TIMED, map(int, out)):
        us = row[4][{0: 0, 1: 1, 2: 2, 3: 3, 5: 4}[tile]]
        if not us or us > 1.06 * min(u for u in row[4] if u):
            bad.append((row, tile))
    assert len(out) == len(TIMED) and not bad, bad
