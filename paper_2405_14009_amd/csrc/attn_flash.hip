// Host side of the fused attention: which shapes it serves, by which kernels.
#include <cmath>

#include "attn_flash.h"
#include "attn_flash_kernels.h"

namespace {

AttnArgs make_args(const void* qkv, int b, int s, int heads, int h) {
  AttnArgs a;
  a.qkv = (const bf16*)qkv;
  a.o = nullptr;
  a.dout = nullptr;
  a.out = nullptr;
  a.lse = nullptr;
  a.dv = nullptr;
  a.s = s;
  a.heads = heads;
  a.bh = b * heads;
  a.h = h;
  a.d = h / heads;
  a.scale = 1.0f / std::sqrt((float)(h / heads));
  a.sl2 = a.scale * 1.4426950408889634f;
  return a;
}

// The paired kernels run one equal-length workgroup per CU.  They are used
// when those workgroups fill the CUs of their last round to 90 % or more, or
// when there are so few that every CU holds at most one anyway (a small
// problem); otherwise the per-block kernels, whose uneven blocks the
// hardware packs two to a CU, lose less to the last round.
bool pair_grid_fills(long wgs) {
  const long cus = device_compute_units();
  if (2 * wgs <= cus) return true;
  const long rounds = (wgs + cus - 1) / cus;
  return 10 * wgs >= 9 * rounds * cus;
}

typedef hipError_t (*Launch)(const AttnArgs&, int, bool, hipStream_t);
// The kernels of the fewest compiled columns that hold the head.
Launch fwd_of(int d) {
  if (d == 128) return attn_fwd_128_full;
  return d <= 32 ? attn_fwd_32 : d <= 64 ? attn_fwd_64 : d <= 96 ? attn_fwd_96 : attn_fwd_128;
}
Launch bwd_of(int d) {
  if (d == 128) return attn_bwd_128_full;
  return d <= 32 ? attn_bwd_32 : d <= 64 ? attn_bwd_64 : d <= 96 ? attn_bwd_96 : attn_bwd_128;
}

bool args_ok(int heads, int h) {
  return heads > 0 && h % heads == 0 && h / heads <= 128 && (h / heads) % 8 == 0;
}

}  // namespace

bool attn_flash_supported(int elt, int head_dim, int s) {
  if (elt != 2 || head_dim > 128 || head_dim % 8) return false;
  return head_dim == 128 || s > 128;
}

bool attn_flash_paired(int b, int s, int heads) {
  const int nqb = (s + 127) / 128;
  return pair_grid_fills((long)((nqb + 1) / 2) * b * heads);
}

hipError_t attn_flash_forward(const void* qkv, void* o, float* lse, int b, int s, int heads, int h,
                              int causal, hipStream_t st) {
  if (!args_ok(heads, h)) return hipErrorInvalidValue;
  if (b <= 0 || s <= 0) return hipSuccess;
  AttnArgs a = make_args(qkv, b, s, heads, h);
  a.out = (bf16*)o;
  a.lse = lse;
  return fwd_of(a.d)(a, causal, attn_flash_paired(b, s, heads), st);
}

hipError_t attn_flash_backward(const void* qkv, const void* o, const void* dout, const float* lse,
                               float* dv_scratch, void* dqkv, int b, int s, int heads, int h, int causal,
                               hipStream_t st) {
  if (!args_ok(heads, h)) return hipErrorInvalidValue;
  if (b <= 0 || s <= 0) return hipSuccess;
  AttnArgs a = make_args(qkv, b, s, heads, h);
  a.o = (const bf16*)o;
  a.dout = (const bf16*)dout;
  a.out = (bf16*)dqkv;
  a.lse = (float*)lse;
  a.dv = dv_scratch;
  return bwd_of(a.d)(a, causal, attn_flash_paired(b, s, heads), st);
}
