// Fused attention kernels of 64 columns (head dimensions up to 64).
#include "attn_flash.h"
#include "attn_flash_kernels.h"

hipError_t attn_fwd_64(const AttnArgs& a, int causal, AttnForm form, hipStream_t st) {
  return attn_fwd_launch<64, false>(a, causal, form, st);
}
hipError_t attn_bwd_64(const AttnArgs& a, int causal, AttnForm form, hipStream_t st) {
  return attn_bwd_launch<64, false>(a, causal, form, st);
}
