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
// one (the operand streams of the CUs compete for the L2s).  `share`: two
// workgroups share a CU and its copy rate, so a round holds twice the CUs, 2 busy
// a k-tile, and `again` counts halves of it.  SHARE_ROUNDS: the workgroups of the
// last round may have a CU each, at `few`, or some of them share one, which sets
// the pace: from `mid` up to the full round's.  SHARE_EVEN: no edges between
// rounds.
enum GemmShare { SHARE_NONE, SHARE_ROUNDS, SHARE_EVEN };
struct GemmCost {
  double fix, again, few, busy;
  GemmShare share;
  double mid;
  double us(long wgs, long ktiles, int cus) const {
    auto kt = [&](double load) { return few + (busy - few) * load * load; };
    const double load = (double)wgs / cus;
    if (share == SHARE_EVEN) return fix + ktiles * std::max(few, busy * load);
    if (share == SHARE_ROUNDS) {
      const long full = wgs / (2L * cus);
      const double rest = load - 2 * full;
      return fix + again * std::max(0.0, load - 1.0) +
             ktiles * (2 * full * busy + (rest <= 0.0 ? 0.0 : rest <= 1.0 ? few : mid + (2 * busy - mid) * (rest - 1.0)));
    }
    const long full = wgs / cus;
    const double rest = load - full;
    return fix + again * (full - (rest > 0.0 ? 0 : 1)) + ktiles * (full * busy + (rest > 0.0 ? kt(rest) : 0.0));
  }
};

// Cost of splitting a bf16 reduction: the launch that sums the partials, a
// thread's walk over them, and their traffic (out and in, and the output).
// Fitted with the tiles' costs below.
inline double split_us(int splits, long M, long N) { return 2.25 + 0.107 * splits + (splits + 1.5) * M * N * 4e-6 / 5.05; }

// bf16 [M, N] product over K (z of them); tn: the weight-gradient layout.
// A CU draws its operands from the L2 at about 47 GB/s whatever the tile, so
// a k-tile of 64 costs about (bm + bn) and the smaller tiles pay for their
// parallelism with operand traffic.  The constants are fits (us) to launches of
// each kernel alone on the card, unsplit and in up to 32 splits, over 1140
// products (M 64 .. 49152, N 64 .. 49152, K 128 .. 49152, drawn over their
// logarithm, grids of 0.25 .. 6 rounds, and the linear layers of h 384 .. 12288
// over 512 .. 16384 tokens), weighted to where a kernel is within 1.1 of the
// fastest.  Weight gradients have their own: their fp32 update adds to every
// round, except in a split, which stores partials.  Over 570 products left out
// of the fit, forward and input gradient / weight gradient, the choice costs on
// average 1.1 % / 0.8 % more than the fastest measured one (3.2 % / 3.7 % with
// fits of fewer shapes, whose partial rounds were too cheap: 1.5 rounds of
// 256x256 tiles over K 12288 take 551 us, three of 256x128 512).
// room_floats: split workspace; colsum_floats: what colsum_rows may take (< 0:
// no column sums).  256x256 tiles unsplit always qualify.
inline GemmPlan plan_bf16(long M, long N, long K, bool tn, long z, long room_floats, long colsum_floats, int cus) {
  struct Kind {
    GemmTile t;
    int bm, bn;
    GemmCost c, ctn;
  };
  static const Kind kinds[6] = {
      {TILE_256, 256, 256, {7.7, 6.5, 1.18, 1.60, SHARE_NONE, 0.0}, {16.7, 20.8, 1.18, 1.66, SHARE_NONE, 0.0}},
      {TILE_256x128, 256, 128, {7.6, 6.3, 0.67, 0.886, SHARE_NONE, 0.0}, {13.5, 13.6, 0.754, 0.962, SHARE_NONE, 0.0}},
      {TILE_128, 128, 128, {4.8, 1.93, 0.754, 0.566, SHARE_ROUNDS, 0.908}, {7.3, 5.3, 0.768, 0.541, SHARE_ROUNDS, 0.874}},
      {TILE_64, 64, 64, {3.34, 0.91, 0.268, 0.25, SHARE_ROUNDS, 0.467}, {4.5, 1.55, 0.333, 0.259, SHARE_ROUNDS, 0.594}},
      {TILE_32, 32, 32, {3.06, 1.54, 0.112, 0.142, SHARE_NONE, 0.0}, {4.05, 1.13, 0.162, 0.212, SHARE_NONE, 0.0}},
      {TILE_192x256, 192, 256, {6.2, 4.4, 0.912, 1.34, SHARE_NONE, 0.0}, {}},
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
      GemmCost c = tn ? q.ctn : q.c;
      if (want > 1) {
        c.fix = q.c.fix;
        c.again = q.c.again;
      }
      double us = c.us(tiles * z * want, q.t == TILE_32 ? (per + 3) / 4 * 4 : per, cus);
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

// Cost of splitting an fp32 reduction: as above, at about 8 TB/s from the caches
// up to 64 MB and 1.25 beyond.
inline double split_f32_us(int splits, long M, long N) {
  const double mb = (splits + 1.5) * M * N * 4e-6;
  return 3.0 + std::min(mb, 64.0) / 8.0 + std::max(0.0, mb - 64.0) / 1.25;
}

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
  static const Kind kinds[3] = {{128, {7.0, 0.0, 2.0, 2.4, SHARE_NONE, 0.0}},
                                {64, {4.7, 0.0, 0.72, 0.57, SHARE_EVEN, 0.0}},
                                {32, {3.3, 2.4, 0.19, 0.19, SHARE_NONE, 0.0}}};
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
      if (want > 1) us += split_f32_us(want, M, N);
      if (us < best_us) {
        best_us = us;
        best = F32Plan{q.b, tiles, want, (int)(per * 32), want > 1 ? want * M * N : 0L};
      }
    }
  }
  return best;
}
