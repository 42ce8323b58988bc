// Launchers of the fused attention kernels by compiled column count (each in a
// translation unit of its own); see attn_flash_kernels.h.
#pragma once

#include <hip/hip_runtime.h>

#include "common.h"
#include "kernels.h"

struct AttnArgs;
#define ATTN_FLASH_DECL(NAME)                                                               \
  hipError_t attn_fwd_##NAME(const AttnArgs& a, int causal, AttnForm form, hipStream_t st); \
  hipError_t attn_bwd_##NAME(const AttnArgs& a, int causal, AttnForm form, hipStream_t st);
ATTN_FLASH_DECL(32)
ATTN_FLASH_DECL(64)
ATTN_FLASH_DECL(96)
ATTN_FLASH_DECL(128)    // head dimensions 104 .. 120
ATTN_FLASH_DECL(128_full)
#undef ATTN_FLASH_DECL
