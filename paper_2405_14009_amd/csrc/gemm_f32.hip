// fp32 GEMM on the fp32 matrix cores (v_mfma_f32_32x32x2_f32: fp32 products
// and sums) for stages stored in fp32.  Same operand conventions, batching,
// causal k-ranges and epilogues as the bf16 family.
//
// What bounds it: at ordinary sizes the matrix cores (256 flop per clock and
// CU, 157 TFLOP/s nominal; a 64x64 tile draws 16 B/clk of operands per CU,
// well below what the L2 delivers); at the smallest sizes the chain of
// k-tiles of the few workgroups that the output has tiles for.  Hence
//   * 64x64 tiles of four waves (one 32x32 MFMA block each), several
//     workgroups per CU, so one's loads hide behind another's products;
//   * k-tiles of 32 through registers into two LDS stages: tile t + 2 is
//     requested while tile t is multiplied, tile t + 1 is written to LDS
//     before the products of tile t, one barrier per k-tile;
//   * reductions split over several workgroups where the output has few tiles.
// LDS layouts.  k-contiguous operand: [row][k], rows padded to 36 floats, so
// the 16-byte fragment reads of 16 consecutive rows fall on distinct banks.
// m/n-contiguous operand: [k][row], k-rows padded by 8 floats, so the two
// half-waves, which read k-rows 4 apart, use different banks.  MFMA e of a
// group of four covers k = 8 g + e (lanes 0-31) and 8 g + 4 + e (lanes 32-63),
// so a lane's four A (and B) values of a group are 4 consecutive k.
#include "gemm.h"
#include "gemm_plan.h"

namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int NT = 256, TK = 32;

// One operand of a k-tile: global -> registers -> LDS.
template <int ROWS, bool KC>
struct Operand {
  static constexpr int STR = KC ? TK + 4 : ROWS + 8;           // floats per LDS row
  static constexpr int FLOATS = KC ? ROWS * STR : TK * STR;    // per stage
  static constexpr int CPR = KC ? TK / 4 : ROWS / 4;           // 16-byte chunks per LDS row
  static constexpr int RPP = NT / CPR;                         // LDS rows per pass
  static constexpr int NP = (KC ? ROWS : TK) / RPP;            // passes
  float4 v[NP];
  int r, c;
  __device__ __forceinline__ void init(int tid) {
    r = tid / CPR;
    c = tid % CPR;
  }
  // rows mn0.. (< MN) and k-range [k0, kend) of the matrix at p; zeros beyond
  __device__ __forceinline__ void load(const float* p, long ld, int mn0, int MN, int k0, int kend) {
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      const int mn = KC ? mn0 + r + RPP * i : mn0 + 4 * c;
      const int k = KC ? k0 + 4 * c : k0 + r + RPP * i;
      v[i] = make_float4(0.f, 0.f, 0.f, 0.f);
      if (mn < MN && k < kend) v[i] = *(const float4*)(p + (KC ? (long)mn * ld + k : (long)k * ld + mn));
    }
  }
  __device__ __forceinline__ void store(float* s) const {
#pragma unroll
    for (int i = 0; i < NP; ++i) *(float4*)(s + (r + RPP * i) * STR + 4 * c) = v[i];
  }
  // the four values of k-group g for row `row` of the tile, half-wave hf
  __device__ __forceinline__ static void frag(const float* s, int row, int g, int hf, float (&f)[4]) {
    if constexpr (KC) {
      const float4 t = *(const float4*)(s + row * STR + 8 * g + 4 * hf);
      f[0] = t.x; f[1] = t.y; f[2] = t.z; f[3] = t.w;
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) f[e] = s[(8 * g + 4 * hf + e) * STR + row];
    }
  }
};

// Workgroup tile 64 WM x 64 WN: 2 x 2 waves of WM x WN MFMA blocks.
template <int WM, int WN, bool AK, bool BKC, int EPI>
__global__ __launch_bounds__(NT) void gemm_f32_kernel(GemmParams p) {
  constexpr int BM = 64 * WM, BN = 64 * WN;
  typedef Operand<BM, AK> OpA;
  typedef Operand<BN, BKC> OpB;
  constexpr int STAGE = OpA::FLOATS + OpB::FLOATS;
  __shared__ __attribute__((aligned(16))) float lds[2 * STAGE];
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
  const int t1 = p.splits > 1 ? min(nk_all, t0 + p.split_k / TK) : nk_all;

  const int tid = threadIdx.x, lane = tid & 63, hf = lane >> 5, col = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  OpA a;
  OpB b;
  a.init(tid);
  b.init(tid);
  auto load = [&](int t) {
    const float* pa = (const float*)p.A;
    const float* pb = (const float*)p.B;
    int k0 = kb + t * TK, kend = ke;
    if (p.kseg_len > 0) {
      const int sg = t / per_seg;
      pa = (const float*)p.segA[sg];
      pb = (const float*)p.segB[sg];
      k0 = (t - sg * per_seg) * TK;
      kend = p.kseg_len;
    }
    a.load(pa + a_off, p.lda, m0, p.M, k0, kend);
    b.load(pb + b_off, p.ldb, n0, p.N, k0, kend);
  };
  f32x16 acc[WM][WN];
#pragma unroll
  for (int i = 0; i < WM; ++i)
#pragma unroll
    for (int j = 0; j < WN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  if (t0 < t1) {
    load(t0);
    a.store(lds);
    b.store(lds + OpA::FLOATS);
    if (t0 + 1 < t1) load(t0 + 1);
  }
  __syncthreads();
  for (int t = t0; t < t1; ++t) {
    const int cur = (t - t0) & 1;
    const float* sa = lds + cur * STAGE;
    const float* sb = sa + OpA::FLOATS;
    if (t + 1 < t1) {  // the other stage was last read before the previous barrier
      float* n = lds + (cur ^ 1) * STAGE;
      a.store(n);
      b.store(n + OpA::FLOATS);
      if (t + 2 < t1) load(t + 2);
    }
#pragma unroll
    for (int g = 0; g < TK / 8; ++g) {
      float fa[WM][4], fb[WN][4];
#pragma unroll
      for (int i = 0; i < WM; ++i) OpA::frag(sa, 32 * (wm * WM + i) + col, g, hf, fa[i]);
#pragma unroll
      for (int j = 0; j < WN; ++j) OpB::frag(sb, 32 * (wn * WN + j) + col, g, hf, fb[j]);
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < WM; ++i)
#pragma unroll
          for (int j = 0; j < WN; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[i][e], fb[j][e], acc[i][j], 0, 0, 0);
    }
    __syncthreads();
  }

  float* C = (float*)p.C + c_off;
#pragma unroll
  for (int i = 0; i < WM; ++i)
#pragma unroll
    for (int j = 0; j < WN; ++j) {
      const f32x16 v = acc[i][j];
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

template <int WM, int WN, bool AK, bool BKC, int EPI>
hipError_t launch(GemmParams p, int splits, int split_k, hipStream_t s) {
  const long tiles = (long)((p.M + 64 * WM - 1) / (64 * WM)) * ((p.N + 64 * WN - 1) / (64 * WN));
  p.splits = splits;
  if (splits == 1) {
    hipLaunchKernelGGL((gemm_f32_kernel<WM, WN, AK, BKC, EPI>), dim3(tiles, p.batch * p.heads), dim3(NT), 0, s, p);
    return hipGetLastError();
  }
  GemmParams q = p;
  q.split_k = split_k;
  q.C = p.split_work;
  q.ldc = p.N;
  hipLaunchKernelGGL((gemm_f32_kernel<WM, WN, AK, BKC, EPI_F32_STORE>), dim3(tiles, splits), dim3(NT), 0, s, q);
  const hipError_t e = hipGetLastError();
  return e != hipSuccess ? e : splitk_finish(4, p, s);
}

template <int WM, int WN, bool AK, bool BKC>
hipError_t launch_epi(const GemmParams& p, hipStream_t s) {
  const bool whole = p.batch * p.heads == 1 && p.krange == KR_FULL && !p.causal_skip;
  const long room = whole && p.split_work ? p.split_floats : 0;
  const SplitPlan pl = plan_f32(p.M, p.N, p.kseg_len > 0 ? p.K / p.kseg_len : 1,
                                p.kseg_len > 0 ? p.kseg_len : p.K, room, device_compute_units());
  switch (p.epi) {
    case EPI_STORE: return launch<WM, WN, AK, BKC, EPI_STORE>(p, pl.splits, pl.split_k, s);
    case EPI_BIAS: return launch<WM, WN, AK, BKC, EPI_BIAS>(p, pl.splits, pl.split_k, s);
    case EPI_BIAS_RESID: return launch<WM, WN, AK, BKC, EPI_BIAS_RESID>(p, pl.splits, pl.split_k, s);
    case EPI_BIAS_GELU: return launch<WM, WN, AK, BKC, EPI_BIAS_GELU>(p, pl.splits, pl.split_k, s);
    case EPI_GELU_BWD: return launch<WM, WN, AK, BKC, EPI_GELU_BWD>(p, pl.splits, pl.split_k, s);
    case EPI_F32_ACC: return launch<WM, WN, AK, BKC, EPI_F32_ACC>(p, pl.splits, pl.split_k, s);
    default: return launch<WM, WN, AK, BKC, EPI_F32_STORE>(p, pl.splits, pl.split_k, s);
  }
}

}  // namespace

GemmWork gemm_f32_work(long M, long N, long nseg, long seg) {
  return {plan_f32(M, N, nseg, seg, GEMM_SPLIT_MAX_FLOATS, 256).split_floats, 0};
}

hipError_t gemm_f32(const GemmParams& p, hipStream_t s) {
  if (p.M <= 0 || p.N <= 0 || p.batch * p.heads <= 0) return hipSuccess;
  if (p.kseg_len > 0 && (p.K % p.kseg_len || p.K / p.kseg_len > GEMM_MAX_SEG || p.krange != KR_FULL))
    return hipErrorInvalidValue;
  // operands are read four elements at a time along their contiguous dimension
  if ((p.a_kcontig ? p.K : p.M) % 4 || (p.b_kcontig ? p.K : p.N) % 4 || p.lda % 4 || p.ldb % 4 ||
      (p.kseg_len > 0 && (p.a_kcontig || p.b_kcontig) && p.kseg_len % 4))
    return hipErrorInvalidValue;
  if (p.colsum_out != nullptr) return hipErrorInvalidValue;  // bf16 products only
  if (p.a_kcontig && !p.b_kcontig) return launch_epi<1, 1, true, false>(p, s);
  if (p.a_kcontig && p.b_kcontig) return launch_epi<1, 1, true, true>(p, s);
  if (!p.a_kcontig && !p.b_kcontig) return launch_epi<1, 1, false, false>(p, s);
  return hipErrorInvalidValue;
}
