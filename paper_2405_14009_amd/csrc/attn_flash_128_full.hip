// Fused attention kernels of head dimension 128.
#include "attn_flash.h"
#include "attn_flash_kernels.h"

hipError_t attn_fwd_128_full(const AttnArgs& a, int causal, AttnForm form, hipStream_t st) {
  return attn_fwd_launch<128, true>(a, causal, form, st);
}
hipError_t attn_bwd_128_full(const AttnArgs& a, int causal, AttnForm form, hipStream_t st) {
  return attn_bwd_launch<128, true>(a, causal, form, st);
}
