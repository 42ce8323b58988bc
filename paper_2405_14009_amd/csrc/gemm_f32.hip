// fp32 GEMM on the fp32 matrix cores (v_mfma_f32_32x32x2_f32: fp32 products
// and sums) for stages stored in fp32.  Same operand conventions, batching,
// causal k-ranges and epilogues as the bf16 family.
//
// What bounds it: the matrix cores (256 flop per clock and CU, 157 TFLOP/s
// nominal) at ordinary sizes, as long as the CU's operand stream keeps up (a
// 64x64 tile draws 16 B/clk per CU at the full rate, which is most of what the
// copies deliver, a 128x128 tile 8); the latency of the k-tile chain of the few
// workgroups there are at the smallest sizes.  Hence 128x128 tiles of eight
// waves where they fill the chip, else 64x64 tiles of four; k-tiles of 32
// copied straight into a ring of LDS stages (buffer-load-to-LDS, up to
// NST - 1 k-tiles in flight, one barrier each); and reductions split over
// several workgroups where the output has few tiles.
// LDS layouts, in 16-byte chunks.  k-contiguous operand: [row][32 k], chunk c
// of row r at c ^ (r / 2 % 8): the fragment reads of 16 consecutive rows fall on
// distinct banks.  m/n-contiguous operand: [k][row], chunk c of k-row k at
// c ^ 8 (k / 4 % 2): the two half-waves, which read k-rows 4 apart, use
// different banks.  MFMA e of a group of four covers k = 8 g + e (lanes 0-31)
// and 8 g + 4 + e (lanes 32-63), so a lane's four A (and B) values of a group
// are 4 consecutive k.
#include "gemm.h"
#include "gemm_plan.h"
#include "gemm_small.h"
#include "mfma_common.h"

namespace {

constexpr int TK = 32;

template <int N>
__device__ __forceinline__ void wait_vm() {  // s_waitcnt vmcnt(N) alone
  __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
}

// One operand of a k-tile: this wave's 1 KB slices (of NW waves) and the
// fragments of one row.
template <int ROWS, bool KC, int NW>
struct Operand {
  static constexpr int BYTES = ROWS * TK * 4;
  static constexpr int ROWB = KC ? TK * 4 : ROWS * 4;  // bytes per LDS row
  static constexpr int CPR = ROWB / 16, RPS = 64 / CPR;
  static constexpr int NI = BYTES / 1024 / NW;
  static_assert(BYTES % (1024 * NW) == 0, "copy split");
  int r, c;  // LDS row of slice 0 and (swizzled back) chunk of this lane
  __device__ __forceinline__ static int swz(int row) { return KC ? (row >> 1) & 7 : ((row >> 2) & 1) << 3; }
  __device__ __forceinline__ void init(int wave, int lane) {
    r = RPS * wave + lane / CPR;
    c = (lane % CPR) ^ swz(r);  // the same for every slice of the wave
  }
  // address of the tile at rows mn0 and k0 of the matrix at p, and the next k-tile's distance
  __device__ __forceinline__ static const float* at(const float* p, long ld, int mn0, int k0) {
    return KC ? p + (long)mn0 * ld + k0 : p + (long)k0 * ld + mn0;
  }
  __device__ __forceinline__ static long step(long ld) { return KC ? TK : TK * ld; }
  // slice q of the tile there: rows mn0.. (< MN), k-range [k0, kend), zeros beyond
  __device__ __forceinline__ void issue(const i32x4& rs, char* tile, long ld, int mn0, int MN, int k0, int kend,
                                        int wave, int q) const {
    const int row = r + RPS * NW * q;
    const bool ok = KC ? (mn0 + row < MN && k0 + 4 * c < kend) : (k0 + row < kend && mn0 + 4 * c < MN);
    const uint32_t off = ok ? (uint32_t)row * (uint32_t)(4 * ld) + 16u * c : kOOB;
    dma16(rs, __builtin_amdgcn_readfirstlane(lds_addr(tile) + (wave + NW * q) * 1024), off);
  }
  // the four values of k-group g for row `row` of the tile, half-wave hf
  __device__ __forceinline__ static void frag(const char* t, int row, int g, int hf, float (&f)[4]) {
    if constexpr (KC) {
      const float4 v = *(const float4*)(t + row * ROWB + (((2 * g + hf) ^ swz(row)) << 4));
      f[0] = v.x; f[1] = v.y; f[2] = v.z; f[3] = v.w;
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int k = 8 * g + 4 * hf + e;  // swz(k) = 8 hf
        f[e] = *(const float*)(t + k * ROWB + (((row >> 2) ^ (hf << 3)) << 4) + 4 * (row & 3));
      }
    }
  }
};

// Workgroup tile 64 WM x 32 WN NWN: 2 x NWN waves of WM x WN MFMA blocks.
template <int WM, int WN, int NWN, int NST, bool AK, bool BKC, int EPI>
__global__ __launch_bounds__(128 * NWN) void gemm_f32_kernel(GemmParams p) {
  constexpr int BM = 64 * WM, BN = 32 * WN * NWN, NW = 2 * NWN;
  typedef Operand<BM, AK, NW> OpA;
  typedef Operand<BN, BKC, NW> OpB;
  constexpr int STAGE = OpA::BYTES + OpB::BYTES, PER_TILE = OpA::NI + OpB::NI;
  __shared__ __attribute__((aligned(1024))) char lds[NST * STAGE];
  const int tiles_m = (p.M + BM - 1) / BM;
  const int tm = blockIdx.x % tiles_m, tn = blockIdx.x / tiles_m;
  const int m0 = tm * BM, n0 = tn * BN;
  if (p.causal_skip && n0 > m0 + BM - 1) return;
  // blockIdx.y: the product of a batch, or the split of a split reduction
  const int split = p.splits > 1 ? blockIdx.y : 0;
  const int z = p.splits > 1 ? 0 : blockIdx.y, zb = z / p.heads, zh = z % p.heads;
  const long a_off = zb * p.a_bs + zh * p.a_hs, b_off = zb * p.b_bs + zh * p.b_hs;
  const long c_off = p.splits > 1 ? (long)split * p.M * p.N : zb * p.c_bs + zh * p.c_hs;
  int kb = 0, ke = p.K;
  if (p.krange == KR_BELOW) ke = min(p.K, m0 + BM);
  else if (p.krange == KR_ABOVE) kb = (m0 / TK) * TK;
  // k-tiles: of one range, or of every segment in turn (a segment's last
  // k-tile is padded with zeros)
  const int per_seg = p.kseg_len > 0 ? (p.kseg_len + TK - 1) / TK : 0;
  const int nk_all = p.kseg_len > 0 ? p.K / p.kseg_len * per_seg : (ke > kb ? (ke - kb + TK - 1) / TK : 0);
  const int t0 = p.splits > 1 ? split * (p.split_k / TK) : 0;
  const int nk = (p.splits > 1 ? min(nk_all, t0 + p.split_k / TK) : nk_all) - t0;

  const int lane = threadIdx.x & 63, hf = lane >> 5, col = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave / NWN, wn = wave % NWN;
  OpA a;
  OpB b;
  a.init(wave, lane);
  b.init(wave, lane);
  // The next k-tile to copy: operand addresses, its k offset in its segment
  // (or the whole range) and that one's end.
  struct {
    const float *a, *b;
    int k0, kend, sg;
  } wk;
  auto at = [&](const void* A, const void* B) {
    wk.a = OpA::at((const float*)A + a_off, p.lda, m0, wk.k0);
    wk.b = OpB::at((const float*)B + b_off, p.ldb, n0, wk.k0);
  };
  wk.sg = 0;
  wk.k0 = kb + t0 * TK;
  wk.kend = ke;
  if (p.kseg_len > 0) {
    wk.sg = t0 / per_seg;
    wk.k0 = (t0 - wk.sg * per_seg) * TK;
    wk.kend = p.kseg_len;
    if (nk > 0) at(p.segA[wk.sg], p.segB[wk.sg]);
  } else {
    at(p.A, p.B);
  }
  auto advance = [&] {
    wk.k0 += TK;
    wk.a += OpA::step(p.lda);
    wk.b += OpB::step(p.ldb);
    if (p.kseg_len > 0 && wk.k0 >= p.kseg_len) {
      wk.k0 = 0;
      ++wk.sg;
      if (wk.sg * per_seg < nk_all) at(p.segA[wk.sg], p.segB[wk.sg]);
    }
  };
  auto issue = [&](char* st, int q) {  // slice q of the PER_TILE of a wave
    if (q < OpA::NI) a.issue(make_rsrc(wk.a, 0x7fffffffL), st, p.lda, m0, p.M, wk.k0, wk.kend, wave, q);
    else b.issue(make_rsrc(wk.b, 0x7fffffffL), st + OpA::BYTES, p.ldb, n0, p.N, wk.k0, wk.kend, wave, q - OpA::NI);
  };
  // Waves of a single block alternate between two accumulators: products that
  // each wait for the one before leave gaps on the matrix core.
  constexpr int NA = WM * WN == 1 ? 2 : 1;
  f32x16 acc[NA][WM][WN];
#pragma unroll
  for (int n = 0; n < NA; ++n)
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
      for (int j = 0; j < WN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[n][i][j][r] = 0.f;

  // Tile i lives in stage i mod NST; iteration i waits for its own copies of
  // tile i and for its fragment reads of tile i - 1, publishes the first and
  // certifies the second with the barrier, requests the fragments of tile i and
  // multiplies tile i - 1 from registers meanwhile, its copies into the stage
  // that tile i - 1 left between the products: with few waves per SIMD the LDS
  // latency and the copies' addresses would otherwise stand between every
  // barrier and its products.
  constexpr int NG = TK / 8;
  static_assert(PER_TILE % NG == 0, "copies between the groups");
  float fa[2][NG][WM][4], fb[2][NG][WN][4];
  auto products = [&](int set, int g) {
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int u = 0; u < WM; ++u)
#pragma unroll
        for (int v = 0; v < WN; ++v)
          acc[e % NA][u][v] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[set][g][u][e], fb[set][g][v][e],
                                                                   acc[e % NA][u][v], 0, 0, 0);
  };
  int sc = 0, si = NST - 1;
  auto step = [&](int i, int set) {
    __builtin_amdgcn_sched_barrier(0);
    if (i + NST - 2 < nk) wait_vm<(NST - 2) * PER_TILE>();
    else wait_vm<0>();
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
    __syncthreads();
    __builtin_amdgcn_sched_barrier(0);
    const char* ta = lds + sc * STAGE;
    const char* tb = ta + OpA::BYTES;
    const bool refill = i + NST - 1 < nk;
    // each group of products with the fragment reads of a group of tile i
    // between them (the last group's go with the one before, so that they are
    // back at the next barrier), then copies
    auto reads = [&](int g) {
#pragma unroll
      for (int q = 0; q < WM; ++q) OpA::frag(ta, 32 * (wm * WM + q) + col, g, hf, fa[set][g][q]);
#pragma unroll
      for (int q = 0; q < WN; ++q) OpB::frag(tb, 32 * (wn * WN + q) + col, g, hf, fb[set][g][q]);
    };
    constexpr int READS = WM * (AK ? 1 : 4) + WN * (BKC ? 1 : 4);  // read instructions of a group
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      __builtin_amdgcn_sched_barrier(0);
      if (i > 0) products(set ^ 1, g);
      if (g < NG - 1) reads(g);
      if (g == NG - 2) reads(NG - 1);
      if (i > 0) {
#pragma unroll
        for (int e = 0; e < 4 * WM * WN; ++e) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x100, (2 * READS + 4 * WM * WN - 1) / (4 * WM * WN), 0);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
      if (refill) {
#pragma unroll
        for (int q = 0; q < PER_TILE / NG; ++q) issue(lds + si * STAGE, g * (PER_TILE / NG) + q);
      }
    }
    if (refill) advance();
    sc = sc + 1 == NST ? 0 : sc + 1;
    si = si + 1 == NST ? 0 : si + 1;
  };
#pragma unroll
  for (int i = 0; i < NST - 1; ++i)
    if (i < nk) {
#pragma unroll
      for (int q = 0; q < PER_TILE; ++q) issue(lds + i * STAGE, q);
      advance();
    }
  for (int i = 0; i < nk; i += 2) {
    step(i, 0);
    if (i + 1 < nk) step(i + 1, 1);
  }
#pragma unroll
  for (int g = 0; g < NG; ++g) {
    if (nk > 0 && (nk & 1)) products(0, g);
    if (nk > 0 && !(nk & 1)) products(1, g);
  }

  float* C = (float*)p.C + c_off;
#pragma unroll
  for (int i = 0; i < WM; ++i)
#pragma unroll
    for (int j = 0; j < WN; ++j) {
      f32x16 v = acc[0][i][j];
      if constexpr (NA > 1) {
#pragma unroll
        for (int r = 0; r < 16; ++r) v[r] += acc[1][i][j][r];
      }
      // lane: column col, rows 8 (r / 4) + 4 hf + r % 4.  The epilogue's inputs
      // of the whole block are requested before its stores.
      const int n = n0 + 32 * (wn * WN + j) + col;
      const int mb = m0 + 32 * (wm * WM + i) + 4 * hf;
      float in[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int m = mb + 8 * (r >> 2) + (r & 3);
        in[r] = 0.f;
        if (n < p.N && m < p.M) {
          if constexpr (EPI == EPI_BIAS_RESID) in[r] = ((const float*)p.resid)[(long)m * p.ld_resid + n];
          if constexpr (EPI == EPI_GELU_BWD) in[r] = ((const float*)p.aux)[(long)m * p.ld_aux + n];
          if constexpr (EPI == EPI_F32_ACC)
            if (p.accumulate) in[r] = C[(long)m * p.ldc + n];
        }
      }
      float bias = 0.f;
      if constexpr (epi_has_bias(EPI))
        if (n < p.N) bias = p.bias[n];
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int m = mb + 8 * (r >> 2) + (r & 3);
        if (n < p.N && m < p.M) {
          const long o = (long)m * p.ldc + n;
          if constexpr (EPI == EPI_BIAS) {
            C[o] = v[r] + bias;
          } else if constexpr (EPI == EPI_BIAS_RESID) {
            C[o] = v[r] + bias + in[r];
          } else if constexpr (EPI == EPI_BIAS_GELU) {
            const float u = v[r] + bias, sg = gelu_sig(u);
            C[o] = gelu_grad_s(u, sg);
            ((float*)p.C2)[(long)m * p.ldc2 + n] = u * sg;
          } else if constexpr (EPI == EPI_GELU_BWD) {
            C[o] = v[r] * in[r];
          } else if constexpr (EPI == EPI_F32_ACC) {
            C[o] = in[r] + v[r];
          } else {
            C[o] = v[r];
          }
        }
      }
    }
}

template <bool AK, bool BKC, int EPI>
hipError_t launch_tiles(const GemmParams& p, const F32Plan& pl, int y, hipStream_t s) {
  const dim3 grid((unsigned)pl.tiles, (unsigned)y);
  if (pl.bm == 128)
    hipLaunchKernelGGL((gemm_f32_kernel<2, 1, 4, 4, AK, BKC, EPI>), grid, dim3(512), 0, s, p);
  else if (pl.bm == 64)
    hipLaunchKernelGGL((gemm_f32_kernel<1, 1, 2, 4, AK, BKC, EPI>), grid, dim3(256), 0, s, p);
  else
    hipLaunchKernelGGL((gemm_small_kernel<float, AK, BKC, EPI>), grid, dim3(256), 0, s, p);
  return hipGetLastError();
}

template <bool AK, bool BKC, int EPI>
hipError_t launch(const GemmParams& p, const F32Plan& pl, hipStream_t s) {
  GemmParams q = p;
  if (f32_wide(p.lda, p.ldb)) {
    q.splits = 1;
    const dim3 grid((unsigned)(((p.M + 31L) / 32) * ((p.N + 31L) / 32)), (unsigned)(p.batch * p.heads));
    hipLaunchKernelGGL((gemm_small_kernel<float, AK, BKC, EPI, true>), grid, dim3(256), 0, s, q);
    return hipGetLastError();
  }
  q.splits = pl.splits;
  if (pl.splits == 1) return launch_tiles<AK, BKC, EPI>(q, pl, p.batch * p.heads, s);
  q.split_k = pl.split_k;
  q.C = p.split_work;
  q.ldc = p.N;
  const hipError_t e = launch_tiles<AK, BKC, EPI_F32_STORE>(q, pl, pl.splits, s);
  if (e != hipSuccess) return e;
  q.C = p.C;
  q.ldc = p.ldc;
  return splitk_finish(4, q, s);
}

template <bool AK, bool BKC>
hipError_t launch_epi(const GemmParams& p, hipStream_t s) {
  const bool whole = p.batch * p.heads == 1 && p.krange == KR_FULL && !p.causal_skip;
  const F32Plan pl = plan_f32(p.M, p.N, p.kseg_len > 0 ? p.K / p.kseg_len : 1, p.kseg_len > 0 ? p.kseg_len : p.K,
                              (long)p.batch * p.heads, whole && p.split_work ? p.split_floats : 0,
                              device_compute_units());
  switch (p.epi) {
    case EPI_STORE: return launch<AK, BKC, EPI_STORE>(p, pl, s);
    case EPI_BIAS: return launch<AK, BKC, EPI_BIAS>(p, pl, s);
    case EPI_BIAS_RESID: return launch<AK, BKC, EPI_BIAS_RESID>(p, pl, s);
    case EPI_BIAS_GELU: return launch<AK, BKC, EPI_BIAS_GELU>(p, pl, s);
    case EPI_GELU_BWD: return launch<AK, BKC, EPI_GELU_BWD>(p, pl, s);
    case EPI_F32_ACC: return launch<AK, BKC, EPI_F32_ACC>(p, pl, s);
    default: return launch<AK, BKC, EPI_F32_STORE>(p, pl, s);
  }
}

}  // namespace

GemmWork gemm_f32_work(long M, long N, long nseg, long seg) {
  return {plan_f32(M, N, nseg, seg, 1, GEMM_SPLIT_MAX_FLOATS, 256).split_floats, 0};
}

hipError_t gemm_f32(const GemmParams& p, hipStream_t s) {
  if (p.M <= 0 || p.N <= 0 || p.batch * p.heads <= 0) return hipSuccess;
  if (p.kseg_len > 0 && (p.K % p.kseg_len || p.K / p.kseg_len > GEMM_MAX_SEG || p.krange != KR_FULL))
    return hipErrorInvalidValue;
  // operands are read four elements at a time along their contiguous dimension
  if ((p.a_kcontig ? p.K : p.M) % 4 || (p.b_kcontig ? p.K : p.N) % 4 || p.lda % 4 || p.ldb % 4 ||
      (p.kseg_len > 0 && (p.a_kcontig || p.b_kcontig) && p.kseg_len % 4))
    return hipErrorInvalidValue;
  if (p.colsum_work != nullptr) return hipErrorInvalidValue;  // bf16 products only
  if (p.a_kcontig && !p.b_kcontig) return launch_epi<true, false>(p, s);
  if (p.a_kcontig && p.b_kcontig) return launch_epi<true, true>(p, s);
  if (!p.a_kcontig && !p.b_kcontig) return launch_epi<false, false>(p, s);
  return hipErrorInvalidValue;
}
