// Fused attention kernels of 128 columns (head dimensions up to 120).
#include "attn_flash.h"
#include "attn_flash_kernels.h"

hipError_t attn_fwd_128(const AttnArgs& a, int causal, AttnForm form, hipStream_t st) {
  return attn_fwd_launch<128, false>(a, causal, form, st);
}
hipError_t attn_bwd_128(const AttnArgs& a, int causal, AttnForm form, hipStream_t st) {
  return attn_bwd_launch<128, false>(a, causal, form, st);
}
