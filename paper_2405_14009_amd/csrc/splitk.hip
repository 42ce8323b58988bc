// Second half of a split GEMM reduction: C = epilogue(sum of the partials).
//
// Bound by memory (the partials come from L2 or the Infinity Cache right
// after their producer): a thread takes four consecutive columns and requests
// the partials of up to eight splits, and the epilogue's input, before it adds
// them in split order, so results do not depend on the launch.  A kernel of
// its own and not the last workgroup of a tile: handing partials from one XCD
// to another inside a launch needs cache write-backs and invalidations per
// workgroup, which cost more than a launch (a 512x1024x4096 product over 64x64
// tiles in two splits: 33.1 us so, 26.6 us unsplit).
#include "gemm.h"

namespace {

template <int EPI, class E>
__global__ __launch_bounds__(256) void splitk_finish_k(GemmParams p) {
  const int nc = p.N / 4;
  const long i = (long)blockIdx.x * 256 + threadIdx.x;
  if (i >= (long)p.M * nc) return;
  const int m = (int)(i / nc), n = 4 * (int)(i % nc);
  const EpiIn<EPI> in = epi_fetch4<EPI, E>(p, p.C, m, n);
  float4 b = make_float4(0.f, 0.f, 0.f, 0.f);
  if constexpr (epi_has_bias(EPI)) b = *(const float4*)(p.bias + n);
  const long mn = (long)p.M * p.N;
  const float* src = p.split_work + (long)m * p.N + n;
  float4 t = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int q0 = 0; q0 < p.splits; q0 += 8) {
    float4 w[8];
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (q0 + u < p.splits) w[u] = *(const float4*)(src + (q0 + u) * mn);
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (q0 + u < p.splits) {
        t.x += w[u].x;
        t.y += w[u].y;
        t.z += w[u].z;
        t.w += w[u].w;
      }
  }
  epi_finish4<EPI, E>(p, p.C, m, n, t, in, b);
}

template <class E>
hipError_t finish(const GemmParams& p, hipStream_t s) {
  const dim3 grid((unsigned)(((long)p.M * (p.N / 4) + 255) / 256));
  switch (p.epi) {
    case EPI_STORE: hipLaunchKernelGGL((splitk_finish_k<EPI_STORE, E>), grid, dim3(256), 0, s, p); break;
    case EPI_BIAS: hipLaunchKernelGGL((splitk_finish_k<EPI_BIAS, E>), grid, dim3(256), 0, s, p); break;
    case EPI_BIAS_RESID: hipLaunchKernelGGL((splitk_finish_k<EPI_BIAS_RESID, E>), grid, dim3(256), 0, s, p); break;
    case EPI_BIAS_GELU: hipLaunchKernelGGL((splitk_finish_k<EPI_BIAS_GELU, E>), grid, dim3(256), 0, s, p); break;
    case EPI_GELU_BWD: hipLaunchKernelGGL((splitk_finish_k<EPI_GELU_BWD, E>), grid, dim3(256), 0, s, p); break;
    case EPI_F32_ACC: hipLaunchKernelGGL((splitk_finish_k<EPI_F32_ACC, E>), grid, dim3(256), 0, s, p); break;
    default: hipLaunchKernelGGL((splitk_finish_k<EPI_F32_STORE, E>), grid, dim3(256), 0, s, p); break;
  }
  return hipGetLastError();
}

}  // namespace

hipError_t splitk_finish(int elt, const GemmParams& p, hipStream_t s) {
  if (p.N % 4) return hipErrorInvalidValue;
  return elt == 2 ? finish<bf16>(p, s) : finish<float>(p, s);
}
