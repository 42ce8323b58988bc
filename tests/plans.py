"""Tile and split of a stage's bf16 products on 256 compute units, from the
library's own rule (gemm_plan.h, compiled for the host), so that a test can
say which kernels its shape runs and fails when a change of the rule moves it."""
import functools
import os
import shutil
import subprocess
import tempfile

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2405_14009_amd", "csrc")
TILES = ("256", "256x128", "128", "64", "32", "192x256")
# The work arena always holds the partials of a stage's best plans (up to 16 Mi
# floats), so the launchers choose as with that much room.
MAIN = r"""
#include <cstdio>
#include <cstdlib>
#include "gemm_plan.h"
int main(int argc, char** argv) {
  const GemmPlan p = plan_bf16(atol(argv[2]), atol(argv[3]), atol(argv[4]), atoi(argv[1]), 1, 16L << 20, -1, 256);
  std::printf("%d %d %ld\n", (int)p.tile, p.splits, p.tiles);
}
"""


@functools.lru_cache(maxsize=None)
def _exe():
    if shutil.which("g++") is None:
        pytest.skip("no host compiler")
    d = tempfile.mkdtemp()
    with open(os.path.join(d, "plan.cpp"), "w") as f:
        f.write(MAIN)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, os.path.join(d, "plan.cpp"), "-o", os.path.join(d, "plan")],
                   check=True)
    return os.path.join(d, "plan")


def product(tn, m, n, k):
    """(tile, splits, kernel) of a product; the persistent kernel takes 256x256
    weight-gradient tiles of more than a round, a multiple of the 8 XCDs."""
    out = subprocess.run([_exe(), str(int(tn)), str(m), str(n), str(k)], capture_output=True, text=True, check=True)
    tile, splits, tiles = map(int, out.stdout.split())
    if tn and tile == 0 and splits == 1 and tiles % 8 == 0 and tiles > 256:
        return "persist", 1
    return TILES[tile], splits


def stage(cfg, n=1):
    """{product: (tile, splits)} of cfg; weight gradients over n micro-batches
    (their tokens padded to whole k-tiles of 64 each)."""
    T, h, f = cfg.tokens, cfg.hidden, cfg.ffn
    k = n * (-(-T // 64) * 64)
    fwd = {"qkv": (3 * h, h), "o": (h, h), "fc1": (f, h), "fc2": (h, f)}
    out = {"f_" + p: product(0, T, a, b) for p, (a, b) in fwd.items()}
    out.update({"d_" + p: product(0, T, b, a) for p, (a, b) in fwd.items()})
    out.update({"w_" + p: product(1, b, a, k) for p, (a, b) in fwd.items()})
    return out
