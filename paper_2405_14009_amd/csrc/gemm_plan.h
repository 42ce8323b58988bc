// Host side of the GEMM launchers: tile and split of the reduction by an
// estimate of the time each choice takes.
#pragma once

#include <algorithm>

enum GemmTile { TILE_256 = 0, TILE_256x128 = 1, TILE_128 = 2, TILE_64 = 3, TILE_32 = 4, TILE_192x256 = 5 };

struct GemmPlan {
  GemmTile tile;
  int bm, bn;
  long tiles;
  int splits, split_k;  // split_k: k per split, a multiple of 64
  long split_floats;    // partials: splits * M * N
  long colsum_rows(long M) const { return (M + bm - 1) / bm * splits; }
};

// A kernel's time: `fix` around its first round of workgroups, `again` around
// every further one, and per k-tile `few` on an empty chip, `busy` on a full
// one (the operand streams of the CUs compete for the L2s).  `two`: two
// workgroups share a CU, and its copy rate, so rounds have no edges.
struct GemmCost {
  double fix, again, few, busy;
  bool two;
  double us(long wgs, long ktiles, int cus) const {
    auto kt = [&](double load) { return few + (busy - few) * load * load; };
    const double load = (double)wgs / cus;
    if (two) return fix + ktiles * std::max(few, busy * load);
    const long full = wgs / cus;
    const double rest = load - full;
    return fix + again * (full - (rest > 0.0 ? 0 : 1)) + ktiles * (full * busy + (rest > 0.0 ? kt(rest) : 0.0));
  }
};

// Cost of splitting a reduction: the launch that sums the partials and its
// traffic (partials out and in, output), which the caches serve at about
// 8 TB/s up to 64 MB; beyond, the partials' store bursts are not hidden
// (2048x4096 in two splits of 256x256 tiles: 62 us for 117 MB).
inline double split_us(int splits, long M, long N) {
  const double mb = (splits + 1.5) * M * N * 4e-6;
  return 3.0 + std::min(mb, 64.0) / 8.0 + std::max(0.0, mb - 64.0) / 1.25;
}

// bf16 [M, N] product over K (z of them); tn: the weight-gradient layout.
// A CU draws its operands from the L2 at about 47 GB/s whatever the tile, so
// a k-tile of 64 costs about (bm + bn) and the smaller tiles pay for their
// parallelism with operand traffic.  The constants are fits (us) to launches
// of each kernel alone on the card, M and N 384 .. 16384, K 384 .. 32768:
// within 10 % where a kernel is the best choice, 30 % elsewhere.
// room_floats: split workspace; colsum_floats: what colsum_rows may take (< 0:
// no column sums).  256x256 tiles unsplit always qualify.
inline GemmPlan plan_bf16(long M, long N, long K, bool tn, long z, long room_floats, long colsum_floats, int cus) {
  struct Kind {
    GemmTile t;
    int bm, bn;
    GemmCost c;
  };
  const Kind kinds[6] = {
      {TILE_256, 256, 256, {14.0, 10.0, 1.09, 1.50, false}},
      {TILE_256x128, 256, 128, {9.8, 2.5, tn ? 0.76 : 0.61, tn ? 1.00 : 0.97, false}},
      {TILE_128, 128, 128, {7.5, 0.0, 0.62, 0.68, true}},
      {TILE_64, 64, 64, {4.0, 0.0, 0.25, 0.28, true}},
      {TILE_32, 32, 32, {3.6, 2.4, 0.07, 0.10, false}},
      {TILE_192x256, 192, 256, {12.0, 3.2, 0.96, 1.31, false}},
  };
  const long nk = std::max(1L, (K + 63) / 64);
  GemmPlan best{};
  double best_us = 1e30;
  for (const Kind& q : kinds) {
    if (tn && q.t == TILE_192x256) continue;  // whole 64-row blocks of a k-contiguous A only
    const long rows = (M + q.bm - 1) / q.bm, tiles = rows * ((N + q.bn - 1) / q.bn);
    for (int want = 1; want <= (q.t == TILE_32 ? 1 : 32); ++want) {
      const long per = (nk + want - 1) / want;
      if ((nk + per - 1) / per != want) continue;  // a split without a k-tile
      if (want > 1 && (per < 2 || want * M * N > room_floats)) break;
      if (colsum_floats >= 0 && (q.t != TILE_256 || want > 1) && rows * want * N > colsum_floats) break;
      // the waves of a 32x32 tile take every fourth k-tile each
      double us = q.c.us(tiles * z * want, q.t == TILE_32 ? (per + 3) / 4 * 4 : per, cus);
      if (want > 1) us += split_us(want, M, N);
      if (us < best_us) {
        best_us = us;
        best = GemmPlan{q.t, q.bm, q.bn, tiles, want, (int)(per * 64), want > 1 ? want * M * N : 0L};
      }
    }
  }
  return best;
}

// Whether an operand of a 128-row tile spans more bytes than the 2^31 that the
// fp32 kernels' buffer offsets reach (tiles start at their own 64-bit address, so
// only the rows of one tile count).  The 32x32 kernel then copies through
// registers; such a stage is bound by its state of tens of GB, not by this.
inline bool f32_wide(long lda, long ldb) { return 127L * 4 * std::max(lda, ldb) + 512 > 0x7fffffffL; }

struct F32Plan {
  int bm;               // tiles of bm x bm: 32, 64 or 128
  long tiles;
  int splits, split_k;  // split_k: k per split, a multiple of 32
  long split_floats;
};

// The same for fp32 products and k-tiles of 32, each segment padded to whole
// k-tiles.  (A 64x64 k-tile takes 0.72 us alone on its CU, 0.57 beside
// another, of which the matrix core needs 0.43; a 128x128 one 2.0 of 1.7.)
inline F32Plan plan_f32(long M, long N, long nseg, long seg, long z, long room_floats, int cus) {
  struct Kind {
    int b;
    GemmCost c;
  };
  static const Kind kinds[3] = {{128, {7.0, 0.0, 2.0, 2.4, false}},
                                {64, {4.7, 0.0, 0.72, 0.57, true}},
                                {32, {3.3, 2.4, 0.19, 0.19, false}}};
  const long nk = std::max(1L, nseg * ((seg + 31) / 32));
  F32Plan best{};
  double best_us = 1e30;
  for (const Kind& q : kinds) {
    const long tiles = ((M + q.b - 1) / q.b) * ((N + q.b - 1) / q.b);
    for (int want = 1; want <= (q.b == 32 ? 1 : 64); ++want) {
      const long per = (nk + want - 1) / want;
      if ((nk + per - 1) / per != want) continue;
      if (want > 1 && (per < 2 || want * M * N > room_floats)) break;
      double us = q.c.us(tiles * z * want, q.b == 32 ? (per + 3) / 4 * 4 : per, cus);
      if (want > 1) us += split_us(want, M, N);
      if (us < best_us) {
        best_us = us;
        best = F32Plan{q.b, tiles, want, (int)(per * 32), want > 1 ? want * M * N : 0L};
      }
    }
  }
  return best;
}
