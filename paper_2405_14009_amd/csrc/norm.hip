// LayerNorm forward / input-gradient kernels (one wave per token row; rows
// too long for one wave take a workgroup), fp32 statistics, wavefront-shuffle
// reductions.
#include "common.h"
#include "kernels.h"

namespace {

constexpr int NT = 256;

template <class E>
__global__ __launch_bounds__(NT) void ln_fwd_k(const E* __restrict__ x, const float* __restrict__ g,
                                               const float* __restrict__ b, E* __restrict__ y,
                                               float* __restrict__ mean, float* __restrict__ rstd,
                                               int h, float eps) {
  __shared__ float red[NT / 64];
  const long row = blockIdx.x;
  const E* xr = x + row * h;
  E* yr = y + row * h;
  float s = 0.f;
  for (int c = threadIdx.x; c < h; c += NT) s += to_f32(xr[c]);
  const float mu = block_sum<NT>(s, red) / h;
  float q = 0.f;
  for (int c = threadIdx.x; c < h; c += NT) {
    const float d = to_f32(xr[c]) - mu;
    q += d * d;
  }
  const float var = block_sum<NT>(q, red) / h;
  const float rs = 1.0f / sqrtf(var + eps);
  for (int c = threadIdx.x; c < h; c += NT) yr[c] = from_f32<E>((to_f32(xr[c]) - mu) * rs * g[c] + b[c]);
  if (threadIdx.x == 0) {
    mean[row] = mu;
    rstd[row] = rs;
  }
}

template <class E>
__global__ __launch_bounds__(NT) void ln_bwd_k(const E* __restrict__ dout, const E* __restrict__ x,
                                               const float* __restrict__ mean,
                                               const float* __restrict__ rstd,
                                               const float* __restrict__ g,
                                               const E* __restrict__ resid, E* __restrict__ dx, int h) {
  __shared__ float red[NT / 64];
  const long row = blockIdx.x;
  const float mu = mean[row], rs = rstd[row];
  const E* dr = dout + row * h;
  const E* xr = x + row * h;
  float s1 = 0.f, s2 = 0.f;
  for (int c = threadIdx.x; c < h; c += NT) {
    const float xh = (to_f32(xr[c]) - mu) * rs;
    const float dz = to_f32(dr[c]) * g[c];
    s1 += dz;
    s2 += dz * xh;
  }
  const float m1 = block_sum<NT>(s1, red) / h;
  const float m2 = block_sum<NT>(s2, red) / h;
  const E* rr = resid + row * h;
  E* out = dx + row * h;
  for (int c = threadIdx.x; c < h; c += NT) {
    const float xh = (to_f32(xr[c]) - mu) * rs;
    const float dz = to_f32(dr[c]) * g[c];
    out[c] = from_f32<E>(to_f32(rr[c]) + rs * (dz - m1 - xh * m2));
  }
}

// ---------------------------------------------------------------------------
// One wave per row with the row held in registers as 16-byte chunks (one HBM
// pass per tensor; MAXC chunks per lane cover rows of up to 64 * MAXC chunks).
template <class E, int MAXC>
__global__ __launch_bounds__(NT) void ln_fwd_wave_k(const E* __restrict__ x, const float* __restrict__ g,
                                                    const float* __restrict__ b, E* __restrict__ y,
                                                    E* __restrict__ xcopy, float* __restrict__ mean,
                                                    float* __restrict__ rstd, long rows, int h, float eps) {
  constexpr int EPC = Chunk<E>::N;
  const long row = blockIdx.x * (long)(NT / 64) + (threadIdx.x >> 6);
  if (row >= rows) return;
  const int lane = threadIdx.x & 63, nc = h / EPC;
  const E* xr = x + row * h;
  uint4 v[MAXC];
  // For rows of up to 8 chunks per lane gamma and beta are requested with the
  // row, not after its reductions (one wave per row and a single round of
  // waves: a later request adds a whole memory round trip to the kernel);
  // longer rows have no registers to spare for them.
  constexpr bool PRE = MAXC <= 8;
  float gg[PRE ? MAXC : 1][EPC], bb[PRE ? MAXC : 1][EPC];
  auto ld_gb = [&](int q, int c, float (&gq)[EPC], float (&bq)[EPC]) {
#pragma unroll
    for (int e = 0; e < EPC; e += 4) {
      *(float4*)(gq + e) = *(const float4*)(g + (long)c * EPC + e);
      *(float4*)(bq + e) = *(const float4*)(b + (long)c * EPC + e);
    }
  };
#pragma unroll
  for (int q = 0; q < MAXC; ++q) {
    const int c = lane + 64 * q;
    if (c < nc) {
      v[q] = *(const uint4*)(xr + (long)c * EPC);
      if constexpr (PRE) ld_gb(q, c, gg[q], bb[q]);
    }
  }
  float s = 0.f;
#pragma unroll
  for (int q = 0; q < MAXC; ++q) {
    if (lane + 64 * q < nc) {
      float f[EPC];
      unpack(v[q], (const E*)nullptr, f);
#pragma unroll
      for (int e = 0; e < EPC; ++e) s += f[e];
    }
  }
  const float mu = wave_sum(s) / h;
  float qv = 0.f;
#pragma unroll
  for (int q = 0; q < MAXC; ++q) {
    if (lane + 64 * q < nc) {
      float f[EPC];
      unpack(v[q], (const E*)nullptr, f);
#pragma unroll
      for (int e = 0; e < EPC; ++e) qv += (f[e] - mu) * (f[e] - mu);
    }
  }
  const float rs = 1.0f / sqrtf(wave_sum(qv) / h + eps);
  E* yr = y + row * h;
#pragma unroll
  for (int q = 0; q < MAXC; ++q) {
    const int c = lane + 64 * q;
    if (c < nc) {
      float f[EPC];
      unpack(v[q], (const E*)nullptr, f);
      const int qi = PRE ? q : 0;
      if constexpr (!PRE) ld_gb(q, c, gg[0], bb[0]);
#pragma unroll
      for (int e = 0; e < EPC; ++e) f[e] = (f[e] - mu) * rs * gg[qi][e] + bb[qi][e];
      *(uint4*)(yr + (long)c * EPC) = pack(f, (const E*)nullptr);
      if (xcopy) *(uint4*)(xcopy + row * h + (long)c * EPC) = v[q];  // the input row, unchanged
    }
  }
  if (lane == 0) {
    mean[row] = mu;
    rstd[row] = rs;
  }
}

template <class E, int MAXC>
__global__ __launch_bounds__(NT) void ln_bwd_wave_k(const E* __restrict__ dout, const E* __restrict__ x,
                                                    const float* __restrict__ mean,
                                                    const float* __restrict__ rstd,
                                                    const float* __restrict__ g,
                                                    const E* __restrict__ resid, E* __restrict__ dx,
                                                    E* __restrict__ rcopy, long rows, int h) {
  constexpr int EPC = Chunk<E>::N;
  const long row = blockIdx.x * (long)(NT / 64) + (threadIdx.x >> 6);
  if (row >= rows) return;
  const int lane = threadIdx.x & 63, nc = h / EPC;
  const float mu = mean[row], rs = rstd[row];
  // For rows of up to 8 chunks per lane every input of the row (the residual
  // and gamma too) is requested before the reductions, so the kernel pays one
  // memory round trip, not two; longer rows load them where they are used.
  constexpr bool PRE = MAXC <= 8;
  uint4 dv[MAXC], xv[MAXC], rv[PRE ? MAXC : 1];
  float gg[PRE ? MAXC : 1][EPC];
  auto ld_g = [&](int c, float (&gq)[EPC]) {
#pragma unroll
    for (int e = 0; e < EPC; e += 4) *(float4*)(gq + e) = *(const float4*)(g + (long)c * EPC + e);
  };
#pragma unroll
  for (int q = 0; q < MAXC; ++q) {
    const int c = lane + 64 * q;
    if (c < nc) {
      dv[q] = *(const uint4*)(dout + row * h + (long)c * EPC);
      xv[q] = *(const uint4*)(x + row * h + (long)c * EPC);
      if constexpr (PRE) {
        rv[q] = *(const uint4*)(resid + row * h + (long)c * EPC);
        ld_g(c, gg[q]);
      }
    }
  }
  float s1 = 0.f, s2 = 0.f;
#pragma unroll
  for (int q = 0; q < MAXC; ++q) {
    const int c = lane + 64 * q;
    if (c < nc) {
      float d[EPC], xx[EPC];
      unpack(dv[q], (const E*)nullptr, d);
      unpack(xv[q], (const E*)nullptr, xx);
      const int qi = PRE ? q : 0;
      if constexpr (!PRE) ld_g(c, gg[0]);
#pragma unroll
      for (int e = 0; e < EPC; ++e) {
        const float dz = d[e] * gg[qi][e];
        s1 += dz;
        s2 += dz * (xx[e] - mu) * rs;
      }
    }
  }
  const float m1 = wave_sum(s1) / h, m2 = wave_sum(s2) / h;
#pragma unroll
  for (int q = 0; q < MAXC; ++q) {
    const int c = lane + 64 * q;
    if (c < nc) {
      float d[EPC], xx[EPC], r[EPC];
      unpack(dv[q], (const E*)nullptr, d);
      unpack(xv[q], (const E*)nullptr, xx);
      const int qi = PRE ? q : 0;
      uint4 rq;
      if constexpr (PRE) {
        rq = rv[q];
      } else {
        rq = *(const uint4*)(resid + row * h + (long)c * EPC);
        ld_g(c, gg[0]);
      }
      unpack(rq, (const E*)nullptr, r);
      if (rcopy) *(uint4*)(rcopy + row * h + (long)c * EPC) = rq;  // the residual row, unchanged
#pragma unroll
      for (int e = 0; e < EPC; ++e) {
        const float xh = (xx[e] - mu) * rs;
        r[e] += rs * (d[e] * gg[qi][e] - m1 - xh * m2);
      }
      *(uint4*)(dx + row * h + (long)c * EPC) = pack(r, (const E*)nullptr);
    }
  }
}

template <class E, int MAXC>
void launch_ln_fwd(const void* x, const float* g, const float* b, void* y, void* xcopy, float* mean,
                   float* rstd, long rows, int h, float eps, hipStream_t s) {
  hipLaunchKernelGGL((ln_fwd_wave_k<E, MAXC>), dim3((unsigned)((rows + 3) / 4)), dim3(NT), 0, s,
                     (const E*)x, g, b, (E*)y, (E*)xcopy, mean, rstd, rows, h, eps);
}
template <class E, int MAXC>
void launch_ln_bwd(const void* dout, const void* x, const float* mean, const float* rstd, const float* g,
                   const void* resid, void* dx, void* rcopy, long rows, int h, hipStream_t s) {
  hipLaunchKernelGGL((ln_bwd_wave_k<E, MAXC>), dim3((unsigned)((rows + 3) / 4)), dim3(NT), 0, s,
                     (const E*)dout, (const E*)x, mean, rstd, g, (const E*)resid, (E*)dx, (E*)rcopy, rows,
                     h);
}

// chunks per lane of a row of h elements of type E, or 0 when the wave
// kernels do not apply (h not a multiple of the chunk, or too long)
int wave_chunks(int elt, int h) {
  const int epc = 16 / elt;
  if (h % epc) return 0;
  const int per = (h / epc + 63) / 64;
  return per <= 24 ? per : 0;
}

}  // namespace

hipError_t ln_forward(int elt, const void* x, const float* g, const float* b, void* y, float* mean,
                      float* rstd, long rows, int h, float eps, hipStream_t s, void* xcopy) {
  if (rows <= 0) return hipSuccess;
  if (const int per = wave_chunks(elt, h)) {
    if (elt == 2) {
      if (per <= 4) launch_ln_fwd<bf16, 4>(x, g, b, y, xcopy, mean, rstd, rows, h, eps, s);
      else if (per <= 8) launch_ln_fwd<bf16, 8>(x, g, b, y, xcopy, mean, rstd, rows, h, eps, s);
      else if (per <= 12) launch_ln_fwd<bf16, 12>(x, g, b, y, xcopy, mean, rstd, rows, h, eps, s);
      else launch_ln_fwd<bf16, 24>(x, g, b, y, xcopy, mean, rstd, rows, h, eps, s);
    } else {
      if (per <= 4) launch_ln_fwd<float, 4>(x, g, b, y, xcopy, mean, rstd, rows, h, eps, s);
      else if (per <= 8) launch_ln_fwd<float, 8>(x, g, b, y, xcopy, mean, rstd, rows, h, eps, s);
      else launch_ln_fwd<float, 24>(x, g, b, y, xcopy, mean, rstd, rows, h, eps, s);
    }
    return hipGetLastError();
  }
  if (xcopy) {  // the row-per-workgroup kernel writes y only
    const hipError_t e = hipMemcpyAsync(xcopy, x, (size_t)rows * h * elt, hipMemcpyDeviceToDevice, s);
    if (e != hipSuccess) return e;
  }
  if (elt == 2)
    hipLaunchKernelGGL(ln_fwd_k<bf16>, dim3(rows), dim3(NT), 0, s, (const bf16*)x, g, b, (bf16*)y,
                       mean, rstd, h, eps);
  else
    hipLaunchKernelGGL(ln_fwd_k<float>, dim3(rows), dim3(NT), 0, s, (const float*)x, g, b,
                       (float*)y, mean, rstd, h, eps);
  return hipGetLastError();
}

hipError_t ln_backward(int elt, const void* dout, const void* x, const float* mean,
                       const float* rstd, const float* g, const void* resid, void* dx, long rows,
                       int h, hipStream_t s, void* rcopy) {
  if (rows <= 0) return hipSuccess;
  if (const int per = wave_chunks(elt, h)) {
    if (elt == 2) {
      if (per <= 4) launch_ln_bwd<bf16, 4>(dout, x, mean, rstd, g, resid, dx, rcopy, rows, h, s);
      else if (per <= 8) launch_ln_bwd<bf16, 8>(dout, x, mean, rstd, g, resid, dx, rcopy, rows, h, s);
      else if (per <= 12) launch_ln_bwd<bf16, 12>(dout, x, mean, rstd, g, resid, dx, rcopy, rows, h, s);
      else launch_ln_bwd<bf16, 24>(dout, x, mean, rstd, g, resid, dx, rcopy, rows, h, s);
    } else {
      if (per <= 4) launch_ln_bwd<float, 4>(dout, x, mean, rstd, g, resid, dx, rcopy, rows, h, s);
      else if (per <= 8) launch_ln_bwd<float, 8>(dout, x, mean, rstd, g, resid, dx, rcopy, rows, h, s);
      else launch_ln_bwd<float, 24>(dout, x, mean, rstd, g, resid, dx, rcopy, rows, h, s);
    }
    return hipGetLastError();
  }
  if (rcopy) {  // the row-per-workgroup kernel writes dx only
    const hipError_t e = hipMemcpyAsync(rcopy, resid, (size_t)rows * h * elt, hipMemcpyDeviceToDevice, s);
    if (e != hipSuccess) return e;
  }
  if (elt == 2)
    hipLaunchKernelGGL(ln_bwd_k<bf16>, dim3(rows), dim3(NT), 0, s, (const bf16*)dout, (const bf16*)x,
                       mean, rstd, g, (const bf16*)resid, (bf16*)dx, h);
  else
    hipLaunchKernelGGL(ln_bwd_k<float>, dim3(rows), dim3(NT), 0, s, (const float*)dout,
                       (const float*)x, mean, rstd, g, (const float*)resid, (float*)dx, h);
  return hipGetLastError();
}
