// GEMM kernel for the smallest outputs, bf16 and fp32: 32x32 tiles, the
// reduction shared by the four waves of the workgroup.
//
// A 64x64 tile leaves a product of a few hundred rows and columns on a few
// dozen compute units, and splitting its reduction over workgroups costs a
// second launch (3 to 4 us, as much as the product).  Here wave w multiplies the
// k-tiles w, w + 4, ... of its workgroup's 32x32 tile with a ring of LDS stages
// of its own (NST of 8 KB, buffer-load-to-LDS): no barrier until the four
// partial tiles are added, in wave order, through LDS.  Bound by the latency of
// a wave's chain of k-tiles.
// LDS layouts, in 16-byte chunks (every operand tile is 4 KB).  k-contiguous:
// 128 bytes per row, chunk c of row r at c ^ (r / 2 % 8).  m/n-contiguous bf16:
// 64 bytes per k-row, in order (the four k-rows of a transposing read are 256
// contiguous bytes).  m/n-contiguous fp32: 128 bytes per k-row, k-row k at row
// k ^ (k / 4 % 2), so that the two half-waves, 4 k-rows apart, use different
// banks.
//
// WIDE: matrices whose 32-row panels span more than the 2^31 bytes that a buffer
// offset reaches (fp32 only; bf16 stages refuse them).  The copies then are
// loads from 64-bit addresses, stored to the same places of the ring.
#pragma once

#include "gemm.h"
#include "mfma_common.h"

namespace {

template <class E, bool KC>
struct SmallOperand {
  static constexpr int BK = 128 / sizeof(E);  // k per k-tile
  static constexpr int EPC = 16 / sizeof(E);  // elements per chunk
  static constexpr int RB = KC || sizeof(E) == 4 ? 128 : 64, CPR = RB / 16, RPS = 64 / CPR;
  // slice q (1 KB, RPS LDS rows) of the k-tile at k0 of the matrix at p: rows
  // mn0.. (< MN), k < kend, zeros beyond
  __device__ __forceinline__ static void issue(const i32x4& rs, char* tile, long ld, int mn0, int MN, int k0,
                                               int kend, int lane, int q) {
    const int r = RPS * q + lane / CPR;
    int mn, k;
    if (KC) {
      mn = r;
      k = EPC * ((lane % CPR) ^ ((r >> 1) & 7));
    } else {
      mn = EPC * (lane % CPR);
      k = sizeof(E) == 4 ? r ^ ((r >> 2) & 1) : r;
    }
    const bool ok = mn0 + mn < MN && k0 + k < kend;
    const uint32_t off = ok ? (uint32_t)(KC ? mn * ld + k : k * ld + mn) * (uint32_t)sizeof(E) : kOOB;
    dma16(rs, __builtin_amdgcn_readfirstlane(lds_addr(tile) + q * 1024), off);
  }
  // the same slice through registers, from p (the matrix at mn0 and k0)
  __device__ __forceinline__ static void copy(const E* p, char* tile, long ld, int mn0, int MN, int k0, int kend,
                                              int lane, int q) {
    const int r = RPS * q + lane / CPR;
    const int mn = KC ? r : EPC * (lane % CPR);
    const int k = KC ? EPC * ((lane % CPR) ^ ((r >> 1) & 7)) : sizeof(E) == 4 ? r ^ ((r >> 2) & 1) : r;
    uint4 v = make_uint4(0, 0, 0, 0);
    if (mn0 + mn < MN && k0 + k < kend) v = *(const uint4*)(p + (KC ? mn * ld + k : k * ld + mn));
    *(uint4*)(tile + q * 1024 + lane * 16) = v;
  }
  __device__ __forceinline__ static const E* at(const E* p, long ld, int mn0, int k0) {
    return KC ? p + (long)mn0 * ld + k0 : p + (long)k0 * ld + mn0;
  }
  __device__ __forceinline__ static long step(long ld) { return KC ? BK : BK * ld; }
};

template <class E> struct SmallFrag;
template <> struct SmallFrag<bf16> { typedef bf16x8 T; };
template <> struct SmallFrag<float> { typedef float4 T; };

// Fragments of the four k-steps of a k-tile for row / column lane % 32.
template <bool KC>
__device__ __forceinline__ void small_frags(const char* t, int lane, bf16x8 (&f)[4]) {
  const int r = lane & 31, hf = lane >> 5;
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) {
    if constexpr (KC) {
      f[ks] = *(const bf16x8*)(t + r * 128 + (((2 * ks + hf) ^ ((r >> 1) & 7)) << 4));
    } else {
      const int i = lane & 15;
      const char* p0 = t + (16 * ks + 8 * hf + (i >> 2)) * 64 + 32 * ((lane >> 4) & 1) + 8 * (i & 3);
      const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t*)p0);
      const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t*)(p0 + 4 * 64));
      f[ks] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    }
  }
}
template <bool KC>
__device__ __forceinline__ void small_frags(const char* t, int lane, float4 (&f)[4]) {
  const int r = lane & 31, hf = lane >> 5;
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    if constexpr (KC) {
      f[g] = *(const float4*)(t + r * 128 + (((2 * g + hf) ^ ((r >> 1) & 7)) << 4));
    } else {
      float v[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = *(const float*)(t + ((8 * g + 4 * hf + e) ^ hf) * 128 + 4 * r);
      f[g] = make_float4(v[0], v[1], v[2], v[3]);
    }
  }
}
__device__ __forceinline__ void small_products(f32x16 (&acc)[2], const bf16x8 (&a)[4], const bf16x8 (&b)[4]) {
#pragma unroll
  for (int ks = 0; ks < 4; ++ks)
    acc[ks & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[ks], b[ks], acc[ks & 1], 0, 0, 0);
}
__device__ __forceinline__ void small_products(f32x16 (&acc)[2], const float4 (&a)[4], const float4 (&b)[4]) {
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    acc[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[g].x, b[g].x, acc[0], 0, 0, 0);
    acc[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[g].y, b[g].y, acc[1], 0, 0, 0);
    acc[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[g].z, b[g].z, acc[0], 0, 0, 0);
    acc[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[g].w, b[g].w, acc[1], 0, 0, 0);
  }
}

template <class E, bool AK, bool BKC, int EPI, bool WIDE = false>
__global__ __launch_bounds__(256) void gemm_small_kernel(GemmParams p) {
  typedef SmallOperand<E, AK> OpA;
  typedef SmallOperand<E, BKC> OpB;
  constexpr int BK = OpA::BK, NST = 4, STAGE = 8192, PER_TILE = 8;
  constexpr int STR = 36;  // floats per row of a partial tile in LDS
  __shared__ __attribute__((aligned(1024))) char lds[4 * NST * STAGE];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  char* const ring = lds + wave * NST * STAGE;
  const int tiles_m = (p.M + 31) / 32;
  const int tm = blockIdx.x % tiles_m, tn = blockIdx.x / tiles_m;
  const int m0 = tm * 32, n0 = tn * 32;
  if (p.causal_skip && n0 > m0 + 31) return;
  const int z = blockIdx.y, zb = z / p.heads, zh = z % p.heads;
  const long a_off = zb * p.a_bs + zh * p.a_hs, b_off = zb * p.b_bs + zh * p.b_hs;
  const long c_off = zb * p.c_bs + zh * p.c_hs;
  int kb = 0, ke = p.K;
  if (p.krange == KR_BELOW) ke = min(p.K, m0 + 32);
  else if (p.krange == KR_ABOVE) kb = (m0 / BK) * BK;
  // k-tiles: of one range, or of every segment in turn (each padded with zeros
  // to whole k-tiles)
  const int per_seg = p.kseg_len > 0 ? (p.kseg_len + BK - 1) / BK : 0;
  const int nseg = p.kseg_len > 0 ? (p.kseg_pad > 0 ? p.K / p.kseg_pad : p.K / p.kseg_len) : 0;
  const int nk_all = nseg > 0 ? nseg * per_seg : (ke > kb ? (ke - kb + BK - 1) / BK : 0);
  const int nk = nk_all > wave ? (nk_all - wave + 3) / 4 : 0;  // this wave's k-tiles

  // the next k-tile of this wave to copy
  int sg = 0, k0 = kb + wave * BK, kend = ke;
  const E *pa = nullptr, *pb = nullptr;
  auto at = [&] {
    if (nseg > 0) {
      pa = OpA::at((const E*)p.segA[sg] + a_off, p.lda, m0, k0);
      pb = OpB::at((const E*)p.segB[sg] + b_off, p.ldb, n0, k0);
    } else {
      pa = OpA::at((const E*)p.A + a_off, p.lda, m0, k0);
      pb = OpB::at((const E*)p.B + b_off, p.ldb, n0, k0);
    }
  };
  auto wrap = [&] {  // into the segment that k0 has run into
    while (k0 >= per_seg * BK && sg < nseg) {
      k0 -= per_seg * BK;
      ++sg;
    }
    if (sg < nseg) at();
  };
  if (nseg > 0) {
    k0 = wave * BK;
    kend = p.kseg_len;
    wrap();
  } else {
    at();
  }
  auto issue = [&](char* st) {
    if constexpr (WIDE) {
#pragma unroll
      for (int q = 0; q < 4; ++q) OpA::copy(pa, st, p.lda, m0, p.M, k0, kend, lane, q);
#pragma unroll
      for (int q = 0; q < 4; ++q) OpB::copy(pb, st + 4096, p.ldb, n0, p.N, k0, kend, lane, q);
    } else {
      const i32x4 ra = make_rsrc(pa, 0x7fffffffL), rb = make_rsrc(pb, 0x7fffffffL);
#pragma unroll
      for (int q = 0; q < 4; ++q) OpA::issue(ra, st, p.lda, m0, p.M, k0, kend, lane, q);
#pragma unroll
      for (int q = 0; q < 4; ++q) OpB::issue(rb, st + 4096, p.ldb, n0, p.N, k0, kend, lane, q);
    }
    k0 += 4 * BK;
    pa += 4 * OpA::step(p.lda);
    pb += 4 * OpB::step(p.ldb);
    if (nseg > 0 && k0 >= per_seg * BK) wrap();
  };

  // Column sums of B (bias gradients, bf16): tile-row tm takes the k-tiles t
  // with t mod tiles_m == tm.  Lane: chunk lane % 4, k-rows lane / 4 + 16 i.
  constexpr bool CS = !AK && !BKC && sizeof(E) == 2;
  const bool cs_on = CS && p.colsum_work != nullptr && z == 0;
  float cs[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) cs[e] = 0.f;

  f32x16 acc[2];
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[0][r] = acc[1][r] = 0.f;
  typename SmallFrag<E>::T fa[2][4], fb[2][4];
  // Iteration i: this wave's copies of its i-th k-tile have landed and its
  // fragment reads of the one before are complete; the stage of that one is
  // refilled, fragments are requested and the one before is multiplied.
  auto step = [&](int i, int set) {
    __builtin_amdgcn_sched_barrier(0);
    if (i + NST - 2 < nk) __builtin_amdgcn_s_waitcnt(0x0070 | ((NST - 2) * PER_TILE & 15) | ((NST - 2) * PER_TILE >> 4 << 14));
    else __builtin_amdgcn_s_waitcnt(0x0070);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    if (i + NST - 1 < nk) issue(ring + (i + NST - 1) % NST * STAGE);
    const char* st = ring + i % NST * STAGE;
    small_frags<AK>(st, lane, fa[set]);
    small_frags<BKC>(st + 4096, lane, fb[set]);
    if constexpr (CS) {
      if (cs_on && (wave + 4 * i) % tiles_m == tm) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const uint4 v = *(const uint4*)(st + 4096 + (lane / 4 + 16 * u) * 64 + (lane & 3) * 16);
          const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            cs[2 * e] += __uint_as_float(w[e] << 16);
            cs[2 * e + 1] += __uint_as_float(w[e] & 0xffff0000u);
          }
        }
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    if (i > 0) small_products(acc, fa[set ^ 1], fb[set ^ 1]);
  };
#pragma unroll
  for (int i = 0; i < NST - 1; ++i)
    if (i < nk) issue(ring + i * STAGE);
  for (int i = 0; i < nk; i += 2) {
    step(i, 0);
    if (i + 1 < nk) step(i + 1, 1);
  }
  if (nk > 0) {
    if (nk & 1) small_products(acc, fa[0], fb[0]);
    else small_products(acc, fa[1], fb[1]);
  }

  // Partial tiles to LDS, each in its wave's own ring (its reads are complete:
  // the products above used them).
  float* const mine = (float*)ring;
#pragma unroll
  for (int r = 0; r < 16; ++r)
    mine[(8 * (r >> 2) + 4 * (lane >> 5) + (r & 3)) * STR + (lane & 31)] = acc[0][r] + acc[1][r];
  constexpr int CS_OFF = 32 * STR;  // floats; then [16 k-row groups][32] column sums
  if constexpr (CS) {
    if (cs_on) {
#pragma unroll
      for (int e = 0; e < 8; ++e) mine[CS_OFF + (lane / 4) * 32 + 8 * (lane & 3) + e] = cs[e];
    }
  }
  __syncthreads();
  const int row = threadIdx.x >> 3, c4 = 4 * (threadIdx.x & 7);
  const int m = m0 + row, n = n0 + c4;
  if (m < p.M && n < p.N) {
    typedef typename EpiOut<EPI, E>::type OutT;
    void* C = (OutT*)p.C + c_off;
    const EpiIn<EPI> in = epi_fetch4<EPI, E>(p, C, m, n);
    float4 bias = make_float4(0.f, 0.f, 0.f, 0.f);
    if constexpr (epi_has_bias(EPI)) bias = *(const float4*)(p.bias + n);
    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const float4 t = *(const float4*)((const float*)(lds + w * NST * STAGE) + row * STR + c4);
      v.x += t.x;
      v.y += t.y;
      v.z += t.z;
      v.w += t.w;
    }
    epi_finish4<EPI, E>(p, C, m, n, v, in, bias);
  }
  if constexpr (CS) {
    if (cs_on && threadIdx.x < 32 && n0 + (int)threadIdx.x < p.N) {
      float t = 0.f;
#pragma unroll
      for (int w = 0; w < 4; ++w)
#pragma unroll
        for (int g = 0; g < 16; ++g) t += ((const float*)(lds + w * NST * STAGE))[CS_OFF + g * 32 + threadIdx.x];
      p.colsum_work[(long)tm * p.N + n0 + threadIdx.x] = t;
    }
  }
}

}  // namespace
