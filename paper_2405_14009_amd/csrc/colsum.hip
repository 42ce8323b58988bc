// Column sums of the weight pass: bias gradients (sums of the output gradients
// over tokens) and LayerNorm-affine gradients, over the tokens of all
// micro-batches of the pass, in a fixed order.
//
// Two launches serve every sum of a layer: partial sums over chunks of rows,
// then the sum of the partial rows (which also takes the partial bias sums that
// the bf16 weight-gradient products leave).  The first is bound by memory: a
// workgroup reads 32 chunks of 16 bytes (512 contiguous bytes) of eight rows at
// a time, eight rows in flight per thread.  Short passes are bound by launches
// and by the rows that one workgroup walks, so chunks shrink from 64 to 16 rows
// until the launch has a workgroup for every compute unit (the reductions of a
// layer at h 1024, 512 tokens took ten launches and 52 us before).
#include <algorithm>

#include "common.h"
#include "kernels.h"

namespace {

constexpr int NT = 256;
constexpr int CW = 32;        // 16-byte chunks per workgroup
constexpr int RG = NT / CW;   // row groups

struct PartArgs {
  ColSegs sg;
  long rows;
  int chunk, cps;             // rows per partial, partials per segment
  int njobs, nchunk;
  struct {
    ColJob j;
    float* part;              // [nchunk][n], LN: gamma's [nchunk][n] after it
    int first;                // first workgroup column of the job
  } job[COLSUM_MAX_JOBS];
};

template <class E>
__global__ __launch_bounds__(NT) void colsum_part_k(PartArgs a) {
  constexpr int EPC = Chunk<E>::N;
  __shared__ float red[2][RG][CW * EPC];
  int ji = 0;
  while (ji + 1 < a.njobs && (int)blockIdx.x >= a.job[ji + 1].first) ++ji;
  const ColJob& j = a.job[ji].j;
  const int cl = threadIdx.x % CW, rg = threadIdx.x / CW;
  const int c0 = ((int)blockIdx.x - a.job[ji].first) * CW * EPC, c = c0 + cl * EPC;
  const int seg = blockIdx.y / a.cps, ch = blockIdx.y % a.cps;
  const char* base = a.sg.base + a.sg.slot[seg] * a.sg.slot_bytes;
  const E* dout = (const E*)(base + j.dout);
  const E* x = (const E*)(base + j.x);
  const float* mean = (const float*)(base + j.mean);
  const float* rstd = (const float*)(base + j.rstd);
  const long r0 = (long)ch * a.chunk, r1 = min(a.rows, r0 + a.chunk);
  float sb[EPC], sg[EPC];
#pragma unroll
  for (int e = 0; e < EPC; ++e) sb[e] = sg[e] = 0.f;
  if (c < j.n) {
    for (long r = r0 + rg; r < r1; r += 8 * RG) {
      uint4 dv[8], xv[8];
      float mu[8], rs[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const long q = r + u * RG;
        if (q < r1) {
          dv[u] = *(const uint4*)(dout + q * j.n + c);
          if (j.ln) {
            xv[u] = *(const uint4*)(x + q * j.n + c);
            mu[u] = mean[q];
            rs[u] = rstd[q];
          }
        }
      }
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (r + u * RG < r1) {
          float d[EPC];
          unpack(dv[u], (const E*)nullptr, d);
#pragma unroll
          for (int e = 0; e < EPC; ++e) sb[e] += d[e];
          if (j.ln) {
            float xx[EPC];
            unpack(xv[u], (const E*)nullptr, xx);
#pragma unroll
            for (int e = 0; e < EPC; ++e) sg[e] += d[e] * (xx[e] - mu[u]) * rs[u];
          }
        }
    }
  }
#pragma unroll
  for (int e = 0; e < EPC; ++e) {
    red[0][rg][cl * EPC + e] = sb[e];
    red[1][rg][cl * EPC + e] = sg[e];
  }
  __syncthreads();
  for (int i = threadIdx.x; i < 2 * CW * EPC; i += NT) {
    const int w = i / (CW * EPC), k = i % (CW * EPC);
    if ((w == 0 || j.ln) && c0 + k < j.n) {
      float t = 0.f;
#pragma unroll
      for (int q = 0; q < RG; ++q) t += red[w][q][k];
      a.job[ji].part[((long)w * a.nchunk + blockIdx.y) * j.n + c0 + k] = t;
    }
  }
}

// out[c] (+)= sum of the rows of src, for several [rows][n] arrays: a workgroup
// takes 64 columns, its 16 row groups every 16th row each, then adds the
// groups in order.
struct FinishArgs {
  int njobs, accumulate;
  struct {
    ColFinish f;
    int first;
  } job[COLSUM_MAX_FINISH];
};
constexpr int FC = 64, FG = NT / (FC / 4);

__global__ __launch_bounds__(NT) void colsum_finish_k(FinishArgs a) {
  __shared__ float4 red[FG][FC / 4];
  int ji = 0;
  while (ji + 1 < a.njobs && (int)blockIdx.x >= a.job[ji + 1].first) ++ji;
  const ColFinish& f = a.job[ji].f;
  const int cl = threadIdx.x % (FC / 4), rg = threadIdx.x / (FC / 4);
  const int c = ((int)blockIdx.x - a.job[ji].first) * FC + 4 * cl;
  float4 t = make_float4(0.f, 0.f, 0.f, 0.f), old = t;
  if (c < f.n) {
    if (rg == 0 && a.accumulate) old = *(const float4*)(f.out + c);
    for (int r = rg; r < f.rows; r += 8 * FG) {
      float4 v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (r + u * FG < f.rows) v[u] = *(const float4*)(f.src + (long)(r + u * FG) * f.n + c);
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (r + u * FG < f.rows) {
          t.x += v[u].x;
          t.y += v[u].y;
          t.z += v[u].z;
          t.w += v[u].w;
        }
    }
  }
  red[rg][cl] = t;
  __syncthreads();
  if (rg == 0 && c < f.n) {
#pragma unroll
    for (int q = 1; q < FG; ++q) {
      const float4 v = red[q][cl];
      t.x += v.x;
      t.y += v.y;
      t.z += v.z;
      t.w += v.w;
    }
    t.x += old.x;
    t.y += old.y;
    t.z += old.z;
    t.w += old.w;
    *(float4*)(f.out + c) = t;
  }
}

int blocks_of(int elt, int n) { return (n + CW * (16 / elt) - 1) / (CW * (16 / elt)); }

// rows per partial for a launch of `cols` workgroup columns
int chunk_rows(long rows, int nseg, int cols) {
  int chunk = 64;
  while (chunk > 16 && (long)nseg * ((rows + chunk - 1) / chunk) * cols < 256) chunk /= 2;
  return chunk;
}

long job_floats(const ColJob& j, int nchunk) { return (j.ln ? 2L : 1L) * nchunk * j.n; }

}  // namespace

long colsum_floats(int elt, const ColJob* jobs, int njobs, int nseg, long rows) {
  int cols = 0;
  for (int i = 0; i < njobs; ++i) cols += blocks_of(elt, jobs[i].n);
  const int chunk = chunk_rows(rows, nseg, cols);
  const int nchunk = nseg * (int)((rows + chunk - 1) / chunk);
  long t = 0;
  for (int i = 0; i < njobs; ++i) t += job_floats(jobs[i], nchunk);
  return t;
}

hipError_t colsum(int elt, const ColSegs& sg, int nseg, long rows, const ColJob* jobs, int njobs,
                  const ColFinish* more, int nmore, int accumulate, float* part, long part_floats, hipStream_t s) {
  if (njobs > COLSUM_MAX_JOBS || nmore > COLSUM_MAX_FINISH) return hipErrorInvalidValue;
  int all = 0;
  for (int i = 0; i < njobs; ++i) {
    if (jobs[i].n % (16 / elt)) return hipErrorInvalidValue;
    all += blocks_of(elt, jobs[i].n);
  }
  int done = 0, donem = 0;
  while (done < njobs || donem < nmore) {
    FinishArgs f;
    f.njobs = 0;
    f.accumulate = accumulate;
    int fcols = 0;
    auto finish = [&](const ColFinish& x) {
      if (x.n % 4) return false;
      f.job[f.njobs].f = x;
      f.job[f.njobs++].first = fcols;
      fcols += (x.n + FC - 1) / FC;
      return true;
    };
    for (; donem < nmore && f.njobs < COLSUM_MAX_FINISH; ++donem)
      if (!finish(more[donem])) return hipErrorInvalidValue;
    // as many jobs as the workspace and the argument tables hold
    PartArgs a;
    a.sg = sg;
    a.rows = rows;
    a.chunk = chunk_rows(rows, nseg, all);
    a.cps = (int)((rows + a.chunk - 1) / a.chunk);
    a.nchunk = nseg * a.cps;
    a.njobs = 0;
    long used = 0;
    int cols = 0;
    while (done < njobs && f.njobs + 2 <= COLSUM_MAX_FINISH) {
      const ColJob& j = jobs[done];
      const long need = job_floats(j, a.nchunk);
      if (used + need > part_floats) {
        if (a.njobs > 0) break;
        if (a.chunk >= 64) return hipErrorInvalidValue;
        a.chunk = 64;
        a.cps = (int)((rows + a.chunk - 1) / a.chunk);
        a.nchunk = nseg * a.cps;
        continue;
      }
      a.job[a.njobs].j = j;
      a.job[a.njobs].part = part + used;
      a.job[a.njobs++].first = cols;
      cols += blocks_of(elt, j.n);
      if (!finish({part + used, a.nchunk, j.n, j.out})) return hipErrorInvalidValue;
      if (j.ln && !finish({part + used + (long)a.nchunk * j.n, a.nchunk, j.n, j.out_g})) return hipErrorInvalidValue;
      used += need;
      ++done;
    }
    if (a.njobs > 0 && a.nchunk > 0) {
      const dim3 grid(cols, a.nchunk);
      if (elt == 2) hipLaunchKernelGGL(colsum_part_k<bf16>, grid, dim3(NT), 0, s, a);
      else hipLaunchKernelGGL(colsum_part_k<float>, grid, dim3(NT), 0, s, a);
      const hipError_t e = hipGetLastError();
      if (e != hipSuccess) return e;
    }
    if (f.njobs == 0) return hipErrorInvalidValue;
    hipLaunchKernelGGL(colsum_finish_k, dim3(fcols), dim3(NT), 0, s, f);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}
