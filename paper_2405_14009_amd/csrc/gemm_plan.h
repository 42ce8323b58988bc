// Host side of the GEMM launchers: tile and split of the reduction by an
// estimate of the time each choice takes.
#pragma once

#include <algorithm>

enum GemmTile { TILE_256 = 0, TILE_256x128 = 1, TILE_128 = 2, TILE_64 = 3 };

struct GemmPlan {
  GemmTile tile;
  int bm, bn;
  long tiles;
  int splits, split_k;  // split_k: k per split, a multiple of 64
  long split_floats;    // partials: splits * M * N
  long colsum_rows(long M) const { return (M + bm - 1) / bm * splits; }
};

// Estimated time (us) of a bf16 [M, N] product over K (z of them): rounds of
// workgroups, each a start and end of `fix` plus its k-tiles of 64 at `kt`; a
// CU draws its operands from the L2 at about 47 GB/s whatever the tile, so kt
// follows (bm + bn) and the smaller tiles pay for their parallelism with more
// operand traffic.  Measured (one box, bf16, us): 256x256 tiles 12.7 + 1.09
// per k-tile with few workgroups, 1.45 with all CUs busy; 256x128 9.8 + 0.61,
// 0.78; 128x128 7.5 + 0.62, 0.70; 64x64 4.4 + 0.275, 0.35 (two share a CU, and
// its copy rate).  A split adds the launch that sums the partials (2 us behind
// its producer) and their traffic at about 4 TB/s.
// room_floats: split workspace; colsum_floats: what colsum_rows may take (< 0:
// no column sums).  256x256 tiles unsplit always qualify.
inline GemmPlan plan_bf16(long M, long N, long K, long z, long room_floats, long colsum_floats, int cus) {
  struct Kind {
    GemmTile t;
    int bm, bn;
    double fix, few, busy;
  };
  static const Kind kinds[4] = {{TILE_256, 256, 256, 12.7, 1.09, 1.45},
                                {TILE_256x128, 256, 128, 9.8, 0.61, 0.78},
                                {TILE_128, 128, 128, 7.5, 0.62, 0.70},
                                {TILE_64, 64, 64, 4.4, 0.275, 0.35}};
  const long nk = std::max(1L, (K + 63) / 64);
  GemmPlan best{};
  double best_us = 1e30;
  for (const Kind& q : kinds) {
    const long tiles = ((M + q.bm - 1) / q.bm) * ((N + q.bn - 1) / q.bn);
    long tried = 0;
    for (int want = 1; want <= 32; ++want) {
      const long per = (nk + want - 1) / want;
      const int splits = (int)((nk + per - 1) / per);  // no split without a k-tile
      if (splits != want || splits == tried) continue;
      tried = splits;
      if (splits > 1 && (per < 2 || (long)splits * M * N > room_floats)) break;
      if (colsum_floats >= 0 && (q.t != TILE_256 || splits > 1) &&
          (M + q.bm - 1) / q.bm * splits * N > colsum_floats)
        break;
      const long wgs = tiles * z * splits;
      const long rounds = (wgs + cus - 1) / cus;
      const double busy = std::min(1.0, (double)wgs / cus);
      const double kt = q.few + (q.busy - q.few) * busy;
      double us = rounds * per * kt + q.fix * (1.0 + 0.25 * (rounds - 1));
      if (splits > 1) us += 2.0 + (splits + 1.5) * M * N * 4e-6 / 4.0;
      if (us < best_us) {
        best_us = us;
        best = GemmPlan{q.t, q.bm, q.bn, tiles, splits, (int)(per * 64),
                        splits > 1 ? (long)splits * M * N : 0L};
      }
    }
  }
  return best;
}

struct F32Plan {
  int bm;               // 64: 64x64 tiles, 128: 128x128
  long tiles;
  int splits, split_k;  // split_k: k per split, a multiple of 32
  long split_floats;
};

// The same for fp32 products over 64x64 or 128x128 tiles and k-tiles of 32,
// each segment padded to whole k-tiles.  Measured (us): 64x64 tiles 4.7 + 0.70
// per k-tile for a workgroup alone on its CU (the matrix core needs 0.43), 0.60
// each for two; 128x128 7 + 2.1 (1.7 needed).
inline F32Plan plan_f32(long M, long N, long nseg, long seg, long z, long room_floats, int cus) {
  struct Kind {
    int b;
    double fix, kt;  // us around a workgroup, per k-tile of a CU's workgroup
  };
  static const Kind kinds[2] = {{128, 7.0, 2.1}, {64, 4.7, 0.70}};
  const long nk = std::max(1L, nseg * ((seg + 31) / 32));
  F32Plan best{};
  double best_us = 1e30;
  for (const Kind& q : kinds) {
    const long tiles = ((M + q.b - 1) / q.b) * ((N + q.b - 1) / q.b);
    for (int want = 1; want <= 64; ++want) {
      const long per = (nk + want - 1) / want;
      if ((nk + per - 1) / per != want) continue;
      if (want > 1 && (per < 2 || want * M * N > room_floats)) break;
      const long rounds = (tiles * z * want + cus - 1) / cus;
      // two 64x64 workgroups share a CU and hide each other's latency
      double us = rounds * per * q.kt * (q.b == 64 && rounds > 1 ? 0.86 : 1.0) + q.fix;
      if (want > 1) us += 2.0 + (want + 1.5) * M * N * 4e-6 / 4.0;
      if (us < best_us) {
        best_us = us;
        best = F32Plan{q.b, tiles, want, (int)(per * 32), want > 1 ? want * M * N : 0L};
      }
    }
  }
  return best;
}
