// bf16 GEMM kernel for outputs that 256-wide tiles leave too few workgroups
// for (128x128 or 64x64 tiles of four waves), and the launcher of all bf16
// products, which picks kernel, tile and split of the reduction.
#pragma once

#include "gemm_bf16_kernel.h"
#include "gemm_plan.h"
#include "gemm_small.h"

namespace {

// One tile (and split) per workgroup of four waves.  The ring of NST stages
// works as in gemm_bf16_kernel: one barrier per k-tile, NST - 1 k-tiles in
// flight.  At these sizes the kernel is bound by the latency of that chain
// (0.25 us per k-tile of 64 for 64x64 tiles with one workgroup per CU, 0.35
// before the multiply ran one k-tile behind the reads), so the ring is as deep
// as two workgroups per CU allow and the launcher splits the reduction until
// the CUs are filled.
template <int BM, int BN, int NST, bool AK, bool BKC, int EPI>
__global__ __launch_bounds__(256) void gemm_bf16_tile_kernel(GemmParams p) {
  static_assert((BM == 128 || BM == 64) && (BN == 128 || BN == 64) && NST >= 2, "tile shapes");
  constexpr int NW = 4, BK = 64, NKS = BK / 16;
  constexpr int TM = BM / 64, TN = BN / 64;  // 32-row blocks per wave
  constexpr int A_BYTES = BM * BK * 2, B_BYTES = BN * BK * 2, STAGE = A_BYTES + B_BYTES;
  constexpr int NIA = A_BYTES / 1024 / NW, NIB = B_BYTES / 1024 / NW;
  constexpr int PER_TILE = NIA + NIB;
  constexpr int EPI_BYTES = 32 * (32 * TN + 8) * 4;
  constexpr int LDS_BYTES = NST * STAGE;
  static_assert(LDS_BYTES <= 160 * 1024 && NW * EPI_BYTES <= LDS_BYTES, "LDS");
  __shared__ __attribute__((aligned(1024))) char lds[LDS_BYTES];

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int tiles_m = (p.M + BM - 1) / BM;
  // consecutive tiles (down a column of tiles, which share a B panel) on one XCD
  const int tile = xcd_tile(blockIdx.x, gridDim.x);
  const int tm = tile % tiles_m, tn = tile / tiles_m;
  const int m0 = tm * BM, n0 = tn * BN;
  if (p.causal_skip && n0 > m0 + BM - 1) return;

  const int split = p.splits > 1 ? blockIdx.y : 0;
  const int z = p.splits > 1 ? 0 : blockIdx.y;
  const int zb = z / p.heads, zh = z % p.heads;
  const long a_off = zb * p.a_bs + zh * p.a_hs, b_off = zb * p.b_bs + zh * p.b_hs;
  const long c_off = p.splits > 1 ? (long)split * p.M * p.N : zb * p.c_bs + zh * p.c_hs;
  int kb = 0, ke = p.K;
  if (p.krange == KR_BELOW) ke = min(p.K, m0 + BM);
  else if (p.krange == KR_ABOVE) kb = (m0 / BK) * BK;
  if (p.splits > 1) {
    kb = split * p.split_k;
    ke = min(p.K, kb + p.split_k);
  }
  const int nk = ke > kb ? (ke - kb + BK - 1) / BK : 0;

  Copier<BM, AK, NIA, NW, BK> ca;
  Copier<BN, BKC, NIB, NW, BK> cb;
  ca.init(wave, p.lda, m0, lane);
  cb.init(wave, p.ldb, n0, lane);
  FragOffsets<BM, AK, TM, NKS, BK> fa;
  FragOffsets<BN, BKC, TN, NKS, BK> fb;
  fa.init(wm * (BM / 2), lane, 0);
  fb.init(wn * (BN / 2), lane, 0);
  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
  // Column sums of B (bias gradients): tile-row tm takes the k-tiles t of its
  // split with t mod tiles_m == tm, into row split * tiles_m + tm.
  constexpr bool CS = !AK && !BKC;
  const bool cs_on = CS && p.colsum_work != nullptr && z == 0;
  int cs_next = tm;
  ColSums<BN, BK, 256> cs;
  if (cs_on) cs.init(threadIdx.x);

  KWalk<AK, BKC, BK> wk;  // the next k-tile to copy
  wk.init(p, a_off, b_off, kb, ke);
  auto issue = [&](char* st) {
    ca.issue(wk.a, st, wave, p.lda, p.M, wk.k, wk.kend);
    cb.issue(wk.b, st + A_BYTES, wave, p.ldb, p.N, wk.k, wk.kend);
    wk.next(p, a_off, b_off);
  };
  // Iteration t waits for its own copies of tile t, publishes them with the
  // barrier, refills the stage of tile t - 1 and requests tile t's fragments.
  // 64x64 tiles (two MFMAs' worth of fragments per k-step and wave) multiply
  // tile t - 1 from registers meanwhile, whose fragment reads must then be
  // complete at the barrier; 128x128 tiles multiply tile t, one k-step behind
  // its reads.
  constexpr bool AHEAD = TM * TN == 1;
  bf16x8 fra[2][AHEAD ? NKS : 1], frb[2][AHEAD ? NKS : 1];
  bf16x8 pa[TM], pb[TN];  // (no deferred products here)
  f32x16 acc2;  // the odd k-steps' sums: products that each wait for the one before leave gaps
  if constexpr (AHEAD) {
#pragma unroll
    for (int r = 0; r < 16; ++r) acc2[r] = 0.f;
  }
  auto products = [&](int set) {
    if constexpr (AHEAD) {
#pragma unroll
      for (int ks = 0; ks < NKS; ks += 2) {
        acc[0][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fra[set][ks], frb[set][ks], acc[0][0], 0, 0, 0);
        acc2 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fra[set][ks + 1], frb[set][ks + 1], acc2, 0, 0, 0);
      }
    }
  };
  int sc = 0, si = NST - 1;
  auto step = [&](int t, int set) {
    __builtin_amdgcn_sched_barrier(0);
    if (t + NST - 2 < nk) wait_vmcnt<(NST - 2) * PER_TILE>();
    else wait_vmcnt<0>();
    if constexpr (AHEAD) __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
    __syncthreads();
    __builtin_amdgcn_sched_barrier(0);
    if (t + NST - 1 < nk) issue(lds + si * STAGE);
    const char* st = lds + sc * STAGE;
    if constexpr (AHEAD) {
#pragma unroll
      for (int ks = 0; ks < NKS; ++ks) {
        fra[set][ks] = frag(st, fa, 0, ks);
        frb[set][ks] = frag(st + A_BYTES, fb, 0, ks);
      }
      __builtin_amdgcn_sched_barrier(0);
      if (t > 0) products(set ^ 1);
    } else {
      mma_tile<BM, BN, AK, BKC, TM, TN, NKS, BK, false>(acc, st, st + A_BYTES, fa, fb, [](int) {}, pa, pb);
    }
    if constexpr (CS) {
      __builtin_amdgcn_sched_barrier(0);
      if (cs_on && t == cs_next) {
        cs.tile(st + A_BYTES);
        cs_next += tiles_m;
      }
    }
    sc = sc + 1 == NST ? 0 : sc + 1;
    si = si + 1 == NST ? 0 : si + 1;
  };
#pragma unroll
  for (int i = 0; i < NST - 1; ++i)
    if (i < nk) issue(lds + i * STAGE);
  for (int t = 0; t < nk; t += 2) {
    step(t, 0);
    if (t + 1 < nk) step(t + 1, 1);
  }
  if constexpr (AHEAD) {
    if (nk > 0) {
      if (nk & 1) products(0);
      else products(1);
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[0][0][r] += acc2[r];
  }
  __builtin_amdgcn_sched_barrier(0);
  __syncthreads();
  static_assert(ColSums<BN, BK, 256>::RED_BYTES <= LDS_BYTES, "column-sum reduction fits LDS");
  if constexpr (CS) {
    if (cs_on) cs.finish((float*)lds, p, split * tiles_m + tm, n0, threadIdx.x);
  }
  epilogue<EPI, TN, 0, TM, true, TM>(p, acc, (float*)(lds + wave * EPI_BYTES), m0 + wm * (BM / 2),
                                     n0 + wn * (BN / 2), lane, c_off);
}

template <bool AK, bool BKC, int EPI>
hipError_t launch_bf16_persist(const GemmParams& p, hipStream_t s) {
  const int ntiles = ((p.M + 255) / 256) * ((p.N + 255) / 256);
  const int per_xcd = std::max(1, device_compute_units() / 8);
  const int nq = std::min(ntiles / 8, per_xcd);
  // Deferred last k-steps (mma_tile) pay off on the long reductions of
  // batched weight gradients (-2 % batched, -7 % for one-round launches), not
  // on single micro-batch ones (+2.4 % at K = 2048).
  if (p.K >= 8192)
    hipLaunchKernelGGL((gemm_bf16_persist_kernel<EPI, AK, BKC, true>), dim3(8 * nq), dim3(512), 0, s, p);
  else
    hipLaunchKernelGGL((gemm_bf16_persist_kernel<EPI, AK, BKC, false>), dim3(8 * nq), dim3(512), 0, s, p);
  return hipGetLastError();
}

// One launch of plan pl over the whole output: grid (tiles, batch or splits).
template <bool AK, bool BKC, int EPI>
hipError_t launch_tiles(const GemmParams& p, const GemmPlan& pl, hipStream_t s) {
  const unsigned y = p.splits > 1 ? (unsigned)p.splits : (unsigned)(p.batch * p.heads);
  const dim3 grid((unsigned)pl.tiles, y);
  switch (pl.tile) {
    case TILE_256:
      // Weight-gradient products of more than one round of tiles run the
      // persistent kernel: each workgroup's next tile starts copying while the
      // previous tile's fp32 gradient update runs (measured on the 6.7B stage's
      // single-micro-batch products: 3-4 % faster; neutral for the forward and
      // input-gradient products, which keep one tile per workgroup).
      if constexpr (!AK && !BKC && EPI != EPI_F32_STORE) {
        if (y == 1 && p.krange == KR_FULL && !p.causal_skip && pl.tiles % 8 == 0 &&
            pl.tiles > device_compute_units())
          return launch_bf16_persist<AK, BKC, EPI>(p, s);
      }
      hipLaunchKernelGGL((gemm_bf16_kernel<256, 256, 8, 1, 64, 2, AK, BKC, EPI>), grid, dim3(512), 0, s, p);
      break;
    case TILE_192x256:
      if constexpr (AK) {
        hipLaunchKernelGGL((gemm_bf16_kernel<192, 256, 8, 1, 64, 2, AK, BKC, EPI>), grid, dim3(512), 0, s, p);
        break;
      }
      return hipErrorInvalidValue;
    case TILE_256x128:
      hipLaunchKernelGGL((gemm_bf16_pp_kernel<128, 2, 3, 4, AK, BKC, EPI>), grid, dim3(512), 0, s, p);
      break;
    case TILE_128:
      hipLaunchKernelGGL((gemm_bf16_tile_kernel<128, 128, 2, AK, BKC, EPI>), grid, dim3(256), 0, s, p);
      break;
    case TILE_64:
      hipLaunchKernelGGL((gemm_bf16_tile_kernel<64, 64, 4, AK, BKC, EPI>), grid, dim3(256), 0, s, p);
      break;
    default:
      hipLaunchKernelGGL((gemm_small_kernel<bf16, AK, BKC, EPI>), grid, dim3(256), 0, s, p);
  }
  return hipGetLastError();
}

template <bool AK, bool BKC, int EPI>
hipError_t launch_bf16(GemmParams p, hipStream_t s) {
  if (p.kseg_len > 0) {  // every segment starts on a k-tile; its last one is padded with zeros
    const int nseg = p.K / p.kseg_len;
    p.kseg_pad = (p.kseg_len + 63) / 64 * 64;
    p.K = nseg * p.kseg_pad;
  }
  const long z = (long)p.batch * p.heads;
  const bool whole = z == 1 && p.krange == KR_FULL && !p.causal_skip;
  const int cus = device_compute_units();
  const GemmPlan pl = plan_bf16(p.M, p.N, p.K, !AK && !BKC, z, whole && p.split_work ? p.split_floats : 0,
                                p.colsum_work != nullptr ? p.colsum_floats : -1, cus);
  if (p.colsum_work != nullptr && pl.colsum_rows(p.M) * p.N > p.colsum_floats) return hipErrorInvalidValue;
  if (p.colsum_work != nullptr) *p.colsum_rows = (int)pl.colsum_rows(p.M);
  p.splits = 1;
  if (pl.splits == 1) return launch_tiles<AK, BKC, EPI>(p, pl, s);
  GemmParams q = p;
  q.splits = pl.splits;
  q.split_k = pl.split_k;
  q.C = p.split_work;
  q.ldc = p.N;
  const hipError_t e = launch_tiles<AK, BKC, EPI_F32_STORE>(q, pl, s);
  if (e != hipSuccess) return e;
  q.C = p.C;
  q.ldc = p.ldc;
  return splitk_finish(2, q, s);
}

}  // namespace
