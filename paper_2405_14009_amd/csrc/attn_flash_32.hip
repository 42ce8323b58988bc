// Fused attention kernels of 32 columns (head dimensions up to 32).
#include "attn_flash.h"
#include "attn_flash_kernels.h"

hipError_t attn_fwd_32(const AttnArgs& a, int causal, AttnForm form, hipStream_t st) {
  return attn_fwd_launch<32, false>(a, causal, form, st);
}
hipError_t attn_bwd_32(const AttnArgs& a, int causal, AttnForm form, hipStream_t st) {
  return attn_bwd_launch<32, false>(a, causal, form, st);
}
