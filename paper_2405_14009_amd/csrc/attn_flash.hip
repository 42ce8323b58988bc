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
  a.orest = nullptr;
  a.lse = nullptr;
  a.dv = nullptr;
  a.s = s;
  a.heads = heads;
  a.bh = b * heads;
  a.rows = (long)b * heads * s;
  a.h = h;
  a.d = h / heads;
  a.scale = 1.0f / std::sqrt((float)(h / heads));
  a.sl2 = a.scale * 1.4426950408889634f;
  return a;
}

// The paired kernels run one workgroup of equal length per CU, the per-block
// ones two or more of uneven length, longest first.  Pairs win only where they
// fill the chip once (us, forward + dQ, pairs / blocks: 32 heads of 128,
// s 2048, 256 pairs, 125 / 134; 16 heads of 64, s 4096, 127 / 159): over
// several rounds the uneven blocks pack better (96 heads of 128, s 2048, 396 /
// 320; 128 heads of 64, s 2048, 299 / 227), and on a part of the chip there
// are more of them (64 heads of 128, s 512, 48 / 38).
bool pair_grid_fills(long wgs) {
  const long cus = device_compute_units();
  return wgs <= cus && 10 * wgs >= 9 * cus;
}

// Whether a grid takes the kernels of small grids: no more workgroups of 32
// rows than compute units hold at once (the tiles of a head of up to 64
// columns let two share a CU).
bool split_grid(int s, int bh, int head_dim) {
  return (long)((s + 31) / 32) * bh <= (head_dim <= 64 ? 2L : 1L) * device_compute_units();
}

typedef hipError_t (*Launch)(const AttnArgs&, int, AttnForm, hipStream_t);
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

// Narrow heads keep the materialised kernels for sequences of one query block.
// They are slower there too (us, one layer, materialised / fused, 16 heads: of 32,
// 64 sequences of 64, 419 / 312; of 64, 8 of 128, 290 / 254; of 96, one of 32,
// 189 / 180), but the fused kernels keep 2 d + 8 bytes per row and head where the
// probabilities take 2 s, so below s = d + 4 a stage would hold more from F to
// B_input than its stash account counts.
bool attn_flash_supported(int elt, int head_dim, int s) {
  if (elt != 2 || head_dim > 128 || head_dim % 8) return false;
  return head_dim == 128 || s > 128;
}

AttnForm attn_flash_form(int b, int s, int heads, int head_dim, int causal) {
  const int nqb = (s + 127) / 128;
  if (split_grid(s, b * heads, head_dim)) return ATTN_SPLIT;
  return causal && pair_grid_fills((long)((nqb + 1) / 2) * b * heads) ? ATTN_PAIRED : ATTN_BLOCK;
}

bool attn_flash_narrow(int head_dim) { return head_dim != 128; }

hipError_t attn_flash_forward(const void* qkv, void* o, void* orest, float* lse, int b, int s, int heads, int h,
                              int causal, hipStream_t st) {
  if (!args_ok(heads, h) || (attn_flash_narrow(h / heads) && !orest)) return hipErrorInvalidValue;
  if (b <= 0 || s <= 0) return hipSuccess;
  AttnArgs a = make_args(qkv, b, s, heads, h);
  a.out = (bf16*)o;
  a.orest = (bf16*)orest;
  a.lse = lse;
  return fwd_of(a.d)(a, causal, attn_flash_form(b, s, heads, a.d, causal), st);
}

hipError_t attn_flash_backward(const void* qkv, const void* o, const void* orest, const void* dout,
                               const float* lse, float* dv_scratch, void* dqkv, int b, int s, int heads, int h,
                               int causal, hipStream_t st) {
  if (!args_ok(heads, h) || (attn_flash_narrow(h / heads) && !orest)) return hipErrorInvalidValue;
  if (b <= 0 || s <= 0) return hipSuccess;
  AttnArgs a = make_args(qkv, b, s, heads, h);
  a.o = (const bf16*)o;
  a.orest = (bf16*)orest;
  a.dout = (const bf16*)dout;
  a.out = (bf16*)dqkv;
  a.lse = (float*)lse;
  a.dv = dv_scratch;
  return bwd_of(a.d)(a, causal, attn_flash_form(b, s, heads, a.d, causal), st);
}
