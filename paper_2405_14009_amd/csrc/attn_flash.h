// Launchers of the fused attention kernels by compiled column count (each in a
// translation unit of its own); see attn_flash_kernels.h.
#pragma once

#include <hip/hip_runtime.h>

#include "common.h"

// Whether a grid takes the kernels of small grids: no more workgroups of 32
// rows than compute units hold at once (the tiles of a head of up to 64
// columns let two share a CU).
inline bool attn_split_grid(int s, int bh, int head_dim) {
  return (long)((s + 31) / 32) * bh <= (head_dim <= 64 ? 2L : 1L) * device_compute_units();
}

struct AttnArgs;
#define ATTN_FLASH_DECL(NAME)                                                              \
  hipError_t attn_fwd_##NAME(const AttnArgs& a, int causal, bool paired, hipStream_t st); \
  hipError_t attn_bwd_##NAME(const AttnArgs& a, int causal, bool paired, hipStream_t st);
ATTN_FLASH_DECL(32)
ATTN_FLASH_DECL(64)
ATTN_FLASH_DECL(96)
ATTN_FLASH_DECL(128)    // head dimensions 104 .. 120
ATTN_FLASH_DECL(128_full)
#undef ATTN_FLASH_DECL
