// Host-side launchers of the non-GEMM stage kernels.  Every launcher
// enqueues on the given stream and returns hipGetLastError().
#pragma once

#include <hip/hip_runtime.h>

// LayerNorm forward over rows of width h: y = (x - mean) * rstd * g + b;
// mean and rstd (fp32) are saved per row.  elt: 2 = bf16, 4 = fp32.  When
// xcopy is given, x is also copied there (rows x h elements).
hipError_t ln_forward(int elt, const void* x, const float* g, const float* b, void* y, float* mean,
                      float* rstd, long rows, int h, float eps, hipStream_t s, void* xcopy = nullptr);

// LayerNorm input gradient plus residual: dx = resid + rstd * (dz - mean(dz)
// - xhat * mean(dz * xhat)), dz = dout * g, xhat recomputed from x, mean, rstd.
// When rcopy is given, resid is also copied there (rows x h elements).
hipError_t ln_backward(int elt, const void* dout, const void* x, const float* mean,
                       const float* rstd, const float* g, const void* resid, void* dx, long rows,
                       int h, hipStream_t s, void* rcopy = nullptr);

// Column sums of one layer's weight pass over the rows of nseg segments (one
// per micro-batch, in the stash slots slot[0..nseg) of slot_bytes each), into
// fp32 outputs (overwrite or accumulate), in a fixed order: partial sums over
// chunks of rows, then their sum.  A job sums a [rows, n] matrix at byte offset
// dout of each segment's slot from base:
//   out[c] (+)= sum_r dout[r, c]
//   ln:   out_g[c] (+)= sum_r dout[r, c] * (x[r, c] - mean[r]) * rstd[r] as well
// n * element size is a multiple of 16.
constexpr int COLSUM_MAX_SEG = 32, COLSUM_MAX_JOBS = 6, COLSUM_MAX_FINISH = 12;
struct ColSegs {
  const char* base;
  size_t slot_bytes;
  int slot[COLSUM_MAX_SEG];
};
struct ColJob {
  size_t dout, x, mean, rstd;
  int n, ln;
  float *out, *out_g;
};
// Partial rows that another kernel left: out[c] (+)= the sum of rows
// src[0..rows)[c].
struct ColFinish {
  const float* src;
  int rows, n;
  float* out;
};
// part (part_floats long) takes the partials; with colsum_floats of it every
// job shares two launches, with that of the largest job alone they take more.
hipError_t colsum(int elt, const ColSegs& segs, int nseg, long rows, const ColJob* jobs, int njobs,
                  const ColFinish* more, int nmore, int accumulate, float* part, long part_floats, hipStream_t s);
long colsum_floats(int elt, const ColJob* jobs, int njobs, int nseg, long rows);

// Attention softmax over materialised scores, rows of length s, z*s rows.
//   forward:  P[r, c] = exp(scale S[r, c] - max) / sum  for c <= q (causal) else 0
//   backward: dS[r, c] = scale * P[r, c] * (dP[r, c] - sum_c' dP P)  (0 where masked)
hipError_t softmax_forward(int elt, const float* S, void* P, long rows, int s, float scale,
                           int causal, hipStream_t st);
hipError_t softmax_backward(int elt, const float* dP, const void* P, void* dS, long rows, int s,
                            float scale, int causal, hipStream_t st);

// Fused attention core (bf16, head dimension d <= 128): per (sequence, head)
// O = softmax(Q K^T / sqrt(d), causal) V without materialising the scores.
// qkv: [b*s, 3h] with column blocks Q | K | V (head j at columns j*d of each);
// o: [b*s, h]; lse: [b, heads, s] fp32 base-2 log-sum-exp of the scaled scores
// (written by the forward, read by the backward), two such arrays for narrow
// heads (attn_flash_narrow): a reference score per row, and log2 of the sum
// relative to it.  The backward writes dQ, dK,
// dV into the three column blocks of dqkv [b*s, 3h]; dv_scratch holds b*heads*s
// floats.  h == heads * d.  orest [b*s, h] (written by the forward, read by the
// backward; narrow heads only): what the bf16 rounding
// of o drops.  Head dimensions other than 128 take it for
// sequences of more than one query block (128).
bool attn_flash_supported(int elt, int head_dim, int s);
// The kernels that fused attention over b sequences of s tokens and `heads`
// heads runs on the current device: one workgroup per query block, per pair of
// query blocks (causal), or per 32 queries, whose waves share their keys.
enum AttnForm { ATTN_BLOCK, ATTN_PAIRED, ATTN_SPLIT };
AttnForm attn_flash_form(int b, int s, int heads, int head_dim, int causal);
bool attn_flash_narrow(int head_dim);  // of the supported ones: not 128
hipError_t attn_flash_forward(const void* qkv, void* o, void* orest, float* lse, int b, int s, int heads, int h,
                              int causal, hipStream_t st);
hipError_t attn_flash_backward(const void* qkv, const void* o, const void* orest, const void* dout,
                               const float* lse, float* dv_scratch, void* dqkv, int b, int s, int heads, int h,
                               int causal, hipStream_t st);

// AdamW over n fp32 parameters; weight decay on indices < n_decay; when wb is
// non-null the first n_decay updated values are also written to it in bf16.
hipError_t adamw_step(float* p, const float* g, float* m, float* v, void* wb, long n, long n_decay,
                      float lr, float beta1, float beta2, float eps, float wd, float step_size,
                      float inv_sqrt_bc2, float grad_scale, hipStream_t s);

// Inverse of adamw_step for the same step number and gradient (rollback);
// first_step != 0 restores the zero initial moments exactly.
hipError_t adamw_undo(float* p, const float* g, float* m, float* v, void* wb, long n, long n_decay,
                      float lr, float beta1, float beta2, float eps, float wd, float step_size,
                      float inv_sqrt_bc2, float grad_scale, int first_step, hipStream_t s);

// Per-block partials over n fp32 gradients (n % 4 == 0): part[b] = sum of
// squares of the finite entries of grad_scale * g, bad[b] = non-finite count,
// for b < GRAD_CHECK_BLOCKS.
constexpr int GRAD_CHECK_BLOCKS = 1024;
hipError_t grad_check(const float* g, long n, float grad_scale, float* part, int* bad, hipStream_t s);

hipError_t cast_f32_to_bf16(const float* src, void* dst, long n, hipStream_t s);
hipError_t fill_f32(float* dst, long n, float value, hipStream_t s);
