// GEMM entry points used by the stage runtime, and the shared epilogue.
//
// C[m, n] = sum_k A(m, k) B(k, n) with
//   A(m, k) = a_kcontig ? A[m*lda + k] : A[k*lda + m]
//   B(k, n) = b_kcontig ? B[n*ldb + k] : B[k*ldb + n]
// so every operand layout of the stage maps onto one kernel family:
//   forward  Y  = X W      : A k-contiguous, B n-contiguous (W stored [in, out])
//   dgrad    dX = dY W^T   : A k-contiguous, B k-contiguous
//   wgrad    dW = X^T dY   : A m-contiguous, B n-contiguous (reduction over tokens)
// Optional batching over z = blockIdx.y in [0, batch*heads) adds
// (z / heads) * *_bs + (z % heads) * *_hs elements to A, B and C (attention).
#pragma once

#include <hip/hip_runtime.h>

#include "common.h"

enum EpiKind {
  EPI_STORE = 0,       // C = acc                                (activation type)
  EPI_BIAS = 1,        // C = acc + bias[n]
  EPI_BIAS_RESID = 2,  // C = acc + bias[n] + resid[m, n]
  EPI_BIAS_GELU = 3,   // u = acc + bias[n];  C = gelu'(u), C2 = gelu(u)
  EPI_GELU_BWD = 4,    // C = acc * aux[m, n]   (aux: the stored gelu'(u))
  EPI_F32_ACC = 5,     // C32 = (accumulate ? C32 : 0) + acc     (fp32 gradient buffers)
  EPI_F32_STORE = 6    // C32 = acc                              (fp32 scores)
};

enum KRange {
  KR_FULL = 0,   // k in [0, K)
  KR_BELOW = 1,  // k < min(K, m0 + BM): operand A is zero for k > m (causal P, dS)
  KR_ABOVE = 2   // k >= m0 rounded down: operand A is zero for k < m (transposed causal P, dS)
};

constexpr int GEMM_MAX_SEG = 32;

struct GemmParams {
  int M, N, K;
  const void* A; long lda; int a_kcontig;
  const void* B; long ldb; int b_kcontig;
  int batch, heads;
  long a_bs, a_hs, b_bs, b_hs, c_bs, c_hs;
  int causal_skip;  // skip output tiles strictly above the diagonal (n0 > m0 + BM - 1)
  int krange;       // KRange
  int epi;          // EpiKind
  void* C; long ldc;
  const float* bias;
  const void* resid; long ld_resid;
  const void* aux; long ld_aux;
  void* C2; long ldc2;
  int accumulate;
  // Column sums of B over k (bf16 GEMMs with A and B m/n-contiguous): the
  // bias gradient of a linear layer is exactly this sum of its output
  // gradient, the B operand of its weight-gradient product.  The workgroup of
  // tile-row tm sums the B tiles it stages anyway whose k-tile index t has
  // t mod tiles_m == tm, into row tm of colsum_work ([rows, N] floats of the
  // colsum_floats there; split s of a split reduction into row
  // s * tiles_m + tm).  Adding up the rows is the caller's (colsum); their
  // number is returned in *colsum_rows.  nullptr: off.
  float* colsum_work;
  long colsum_floats;
  int* colsum_rows;
  // Split reductions: with splits > 1 (set by the launchers, which also point
  // C at the partials) workgroup row blockIdx.y multiplies k in
  // [y * split_k, (y + 1) * split_k) and stores its fp32 partial of the whole
  // [M, N] output at C + y * M * N; splitk_finish then adds the partials in
  // order and runs the epilogue.  The launchers split where it pays and
  // split_floats of workspace at split_work (nullptr: none) allow it.
  float* split_work;
  long split_floats;
  int splits, split_k;
  // Reduction split into segments of kseg_len (0: one segment).  Segment s
  // of A / B starts at segA[s] / segB[s] (A, B are ignored); within a segment
  // the layouts above apply with k counted from the segment start.  Used to
  // run several micro-batches' weight gradients as one product over their
  // concatenated tokens.
  int kseg_len;
  int kseg_pad;  // set by the bf16 launcher: kseg_len rounded up to whole k-tiles, K counts padded segments
  const void* segA[GEMM_MAX_SEG];
  const void* segB[GEMM_MAX_SEG];
};

// Shapes must satisfy: M, N, K multiples of 8 when an operand is loaded
// along that dimension in 8-element vectors (checked by the caller).
hipError_t gemm_bf16(const GemmParams& p, hipStream_t s);
// Workspace of a product of [M, N] over nseg segments of seg each: floats of
// split_work that it can make use of, and of colsum_work that column sums need.
struct GemmWork {
  long split_floats, colsum_floats;
};
GemmWork gemm_bf16_work(long M, long N, long nseg, long seg, bool tn);  // tn: A and B m/n-contiguous
GemmWork gemm_f32_work(long M, long N, long nseg, long seg);
constexpr long GEMM_SPLIT_MAX_FLOATS = 16L << 20;  // most partials of one product
hipError_t gemm_f32(const GemmParams& p, hipStream_t s);

// Per-element input of an epilogue at (m, n..n+3): the residual, GeLU's
// input, or the fp32 gradient being accumulated into.  Fetched separately
// from the arithmetic so that a tile's epilogue can have a whole block-row of
// these loads in flight instead of one load round trip per output group.
template <int EPI>
struct EpiIn {
  static constexpr bool kHas = EPI == EPI_BIAS_RESID || EPI == EPI_GELU_BWD || EPI == EPI_F32_ACC;
  uint4 raw;
};

template <int EPI, class E>
__device__ __forceinline__ EpiIn<EPI> epi_fetch4(const GemmParams& p, const void* Cv, int m, int n) {
  EpiIn<EPI> r;
  r.raw = make_uint4(0, 0, 0, 0);
  auto ld = [](const E* q) -> uint4 {
    if constexpr (sizeof(E) == 2) {
      const uint2 u = *(const uint2*)q;
      return make_uint4(u.x, u.y, 0, 0);
    } else {
      return *(const uint4*)q;
    }
  };
  if constexpr (EPI == EPI_BIAS_RESID) {
    r.raw = ld((const E*)p.resid + (long)m * p.ld_resid + n);
  } else if constexpr (EPI == EPI_GELU_BWD) {
    r.raw = ld((const E*)p.aux + (long)m * p.ld_aux + n);
  } else if constexpr (EPI == EPI_F32_ACC) {
    if (p.accumulate) r.raw = *(const uint4*)((const float*)Cv + (long)m * p.ldc + n);
  }
  return r;
}

constexpr bool epi_has_bias(int epi) {
  return epi == EPI_BIAS || epi == EPI_BIAS_RESID || epi == EPI_BIAS_GELU;
}

// The epilogue on 4 consecutive columns n..n+3 (n % 4 == 0, all in range)
// given their fetched input and bias[n..n+3] (loaded once by the caller: a
// lane's columns are the same on every row); 8- or 16-byte vector stores.
template <int EPI, class E>
__device__ __forceinline__ void epi_finish4(const GemmParams& p, void* Cv, int m, int n, float4 v,
                                            const EpiIn<EPI>& in, float4 b) {
  const long i = (long)m * p.ldc + n;
  auto cvt4 = [](uint4 u) -> float4 {
    if constexpr (sizeof(E) == 2) {
      return make_float4(__uint_as_float(u.x << 16), __uint_as_float(u.x & 0xffff0000u),
                         __uint_as_float(u.y << 16), __uint_as_float(u.y & 0xffff0000u));
    } else {
      return make_float4(__uint_as_float(u.x), __uint_as_float(u.y), __uint_as_float(u.z),
                         __uint_as_float(u.w));
    }
  };
  auto st4 = [](E* q, float4 f) {
    if constexpr (sizeof(E) == 2) {
      E t[4] = {from_f32<E>(f.x), from_f32<E>(f.y), from_f32<E>(f.z), from_f32<E>(f.w)};
      *(uint2*)q = *(const uint2*)t;
    } else {
      *(float4*)q = f;
    }
  };
  if constexpr (EPI == EPI_F32_ACC) {
    if (p.accumulate) {
      v.x += __uint_as_float(in.raw.x); v.y += __uint_as_float(in.raw.y);
      v.z += __uint_as_float(in.raw.z); v.w += __uint_as_float(in.raw.w);
    }
    *(float4*)((float*)Cv + i) = v;
  } else if constexpr (EPI == EPI_F32_STORE) {
    *(float4*)((float*)Cv + i) = v;
  } else {
    E* C = (E*)Cv;
    if constexpr (epi_has_bias(EPI)) {
      v.x += b.x; v.y += b.y; v.z += b.z; v.w += b.w;
    }
    if constexpr (EPI == EPI_BIAS_RESID) {
      const float4 r = cvt4(in.raw);
      v.x += r.x; v.y += r.y; v.z += r.z; v.w += r.w;
    }
    if constexpr (EPI == EPI_GELU_BWD) {
      const float4 d = cvt4(in.raw);
      v.x *= d.x; v.y *= d.y; v.z *= d.z; v.w *= d.w;
    }
    if constexpr (EPI == EPI_BIAS_GELU) {
      const float4 sg = make_float4(gelu_sig(v.x), gelu_sig(v.y), gelu_sig(v.z), gelu_sig(v.w));
      st4(C + i, make_float4(gelu_grad_s(v.x, sg.x), gelu_grad_s(v.y, sg.y), gelu_grad_s(v.z, sg.z),
                             gelu_grad_s(v.w, sg.w)));
      st4((E*)p.C2 + (long)m * p.ldc2 + n, make_float4(v.x * sg.x, v.y * sg.y, v.z * sg.z, v.w * sg.w));
    } else {
      st4(C + i, v);
    }
  }
}

// Output element type of each epilogue given the activation type E.
template <int EPI, class E>
struct EpiOut { typedef E type; };
template <class E> struct EpiOut<EPI_F32_ACC, E> { typedef float type; };
template <class E> struct EpiOut<EPI_F32_STORE, E> { typedef float type; };

// Adds the partials of a split reduction in order and runs the epilogue of p
// (whose C is the output again).
hipError_t splitk_finish(int elt, const GemmParams& p, hipStream_t s);
