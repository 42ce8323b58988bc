// bf16 GEMMs with A k-contiguous and B n-contiguous (forward Y = X W, and
// the attention products P V and dS K), plus the top-level bf16 dispatcher.
#include "gemm_bf16_tile.h"

hipError_t gemm_bf16_nt(const GemmParams& p, hipStream_t s);
hipError_t gemm_bf16_tn(const GemmParams& p, hipStream_t s);

static hipError_t gemm_bf16_nn(const GemmParams& p, hipStream_t s) {
  switch (p.epi) {
    case EPI_STORE: return launch_bf16<true, false, EPI_STORE>(p, s);
    case EPI_BIAS: return launch_bf16<true, false, EPI_BIAS>(p, s);
    case EPI_BIAS_RESID: return launch_bf16<true, false, EPI_BIAS_RESID>(p, s);
    case EPI_BIAS_GELU: return launch_bf16<true, false, EPI_BIAS_GELU>(p, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t gemm_bf16(const GemmParams& p, hipStream_t s) {
  if (p.M <= 0 || p.N <= 0 || p.batch * p.heads <= 0) return hipSuccess;
  // only weight-gradient products are segmented
  if (p.kseg_len > 0 && (p.K % p.kseg_len || p.K / p.kseg_len > GEMM_MAX_SEG || p.krange != KR_FULL ||
                         p.a_kcontig || p.b_kcontig))
    return hipErrorInvalidValue;
  if (p.a_kcontig && !p.b_kcontig) return gemm_bf16_nn(p, s);
  // column sums of B: weight-gradient layout only, with its workspace
  if (p.colsum_work != nullptr && (p.a_kcontig || p.b_kcontig || p.colsum_rows == nullptr || p.batch * p.heads != 1))
    return hipErrorInvalidValue;
  if (p.a_kcontig && p.b_kcontig) return gemm_bf16_nt(p, s);
  if (!p.a_kcontig && !p.b_kcontig) return gemm_bf16_tn(p, s);
  return hipErrorInvalidValue;
}

GemmWork gemm_bf16_work(long M, long N, long nseg, long seg, bool tn) {
  // sized for 256 compute units; on a device with others the launcher splits
  // within that room
  const GemmPlan pl =
      plan_bf16(M, N, nseg * ((seg + 63) / 64) * 64, tn, 1, GEMM_SPLIT_MAX_FLOATS, -1, 256);
  return {pl.split_floats, std::max(pl.colsum_rows(M), (M + 255) / 256) * N};
}
