// Fused attention kernels of 96 columns (head dimensions up to 96).
#include "attn_flash.h"
#include "attn_flash_kernels.h"

hipError_t attn_fwd_96(const AttnArgs& a, int causal, AttnForm form, hipStream_t st) {
  return attn_fwd_launch<96, false>(a, causal, form, st);
}
hipError_t attn_bwd_96(const AttnArgs& a, int causal, AttnForm form, hipStream_t st) {
  return attn_bwd_launch<96, false>(a, causal, form, st);
}
