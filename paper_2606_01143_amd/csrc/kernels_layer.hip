// Token-wise operations of a decoder layer: RMSNorm, rotary embedding and
// SwiGLU, forward and backward.  Each streams its tensors once with 16-byte
// accesses (HBM bound); reductions of a row stay inside one workgroup.
#include <math.h>

#include "launch.hpp"

namespace spr {

namespace {
constexpr int kRowThreads = 256;

__device__ __forceinline__ void load8(const bf16* p, float (&v)[8]) {
  const bf16x8 x = *(const bf16x8*)p;
#pragma unroll
  for (int j = 0; j < 8; ++j) v[j] = (float)x[j];
}
__device__ __forceinline__ void store8(bf16* p, const float (&v)[8]) {
  bf16x8 x;
#pragma unroll
  for (int j = 0; j < 8; ++j) x[j] = (bf16)v[j];
  *(bf16x8*)p = x;
}

// sum over the workgroup, the same value returned to every thread
__device__ float block_sum(float v, float* red) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  __syncthreads();
  if (lane == 0) red[w] = v;
  __syncthreads();
  float s = 0.f;
  for (int i = 0; i < kRowThreads / 64; ++i) s += red[i];
  return s;
}
}  // namespace

// one workgroup per row; each thread holds up to 8 chunks of 8 values
constexpr int kMaxChunks = 8;

__global__ __launch_bounds__(kRowThreads) void rmsnorm_fwd_kernel(const bf16* __restrict__ x, bf16* __restrict__ y,
                                                                  float* __restrict__ rstd, int width, float eps) {
  __shared__ float red[kRowThreads / 64];
  const long row = blockIdx.x;
  const bf16* xr = x + row * width;
  const int chunks = width / 8;
  float v[kMaxChunks][8];
  float ss = 0.f;
#pragma unroll
  for (int c = 0; c < kMaxChunks; ++c) {
    const int ch = threadIdx.x + c * kRowThreads;
    if (ch < chunks) {
      load8(xr + 8 * ch, v[c]);
#pragma unroll
      for (int j = 0; j < 8; ++j) ss = fmaf(v[c][j], v[c][j], ss);
    }
  }
  const float r = rsqrtf(block_sum(ss, red) / (float)width + eps);
#pragma unroll
  for (int c = 0; c < kMaxChunks; ++c) {
    const int ch = threadIdx.x + c * kRowThreads;
    if (ch < chunks) {
      float o[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) o[j] = v[c][j] * r;
      store8(y + row * width + 8 * ch, o);
    }
  }
  if (threadIdx.x == 0) rstd[row] = r;
}

__global__ __launch_bounds__(kRowThreads) void rmsnorm_bwd_kernel(const bf16* __restrict__ x,
                                                                  const float* __restrict__ rstd,
                                                                  const bf16* __restrict__ dy,
                                                                  const bf16* __restrict__ add, bf16* __restrict__ dx,
                                                                  int width) {
  __shared__ float red[kRowThreads / 64];
  const long row = blockIdx.x;
  const int chunks = width / 8;
  const float r = rstd[row];
  float xv[kMaxChunks][8], gv[kMaxChunks][8];
  float dot = 0.f;
#pragma unroll
  for (int c = 0; c < kMaxChunks; ++c) {
    const int ch = threadIdx.x + c * kRowThreads;
    if (ch < chunks) {
      load8(x + row * width + 8 * ch, xv[c]);
      load8(dy + row * width + 8 * ch, gv[c]);
#pragma unroll
      for (int j = 0; j < 8; ++j) dot = fmaf(gv[c][j], xv[c][j], dot);
    }
  }
  // dx = r dy - r^3 x mean(dy x)
  const float k3 = r * r * r * block_sum(dot, red) / (float)width;
#pragma unroll
  for (int c = 0; c < kMaxChunks; ++c) {
    const int ch = threadIdx.x + c * kRowThreads;
    if (ch < chunks) {
      float o[8], a[8];
      if (add)
        load8(add + row * width + 8 * ch, a);
      else
#pragma unroll
        for (int j = 0; j < 8; ++j) a[j] = 0.f;
#pragma unroll
      for (int j = 0; j < 8; ++j) o[j] = r * gv[c][j] - k3 * xv[c][j] + a[j];
      store8(dx + row * width + 8 * ch, o);
    }
  }
}

// cos and sin of token position pos at frequency theta^(-2j/d): angle in
// fp64, reduced to [-pi, pi] before the fp32 sine and cosine
__device__ __forceinline__ float2 rope_angle(double pos, double freq, float sign) {
  const double ang = remainder(pos * freq, 2.0 * M_PI);
  float sn, cs;
  sincosf((float)ang, &sn, &cs);
  return make_float2(cs, sn * sign);
}

// head dims that are a multiple of 16 (16-byte chunks of both halves): one
// workgroup per kRopeTokens tokens.  The fp64 power, reduction and sincos of
// a pair (token, j) cost far more than the memory the pair moves, and are the
// same for every head, so each is computed once into LDS and the heads
// stream past it; the first kRopeAhead chunk pairs of a thread are loaded
// before the angles are formed.  Measured on 4096 tokens x 32 heads x 128
// (67 MB): one angle per (token, head, j) 87 us, this form 14.4 us
// (4.7 TB/s).
constexpr int kRopeTokens = 4, kRopeAhead = 4, kRopeMaxHalf = 128;

__global__ __launch_bounds__(kRowThreads) void rope_shared_kernel(const bf16* x, bf16* y, long tokens, int heads,
                                                                  int d, int pos0, double theta, float sign) {
  __shared__ float2 cs[kRopeTokens][kRopeMaxHalf];
  const int half = d / 2, cpr = half / 8;  // 16-byte chunks per half row
  const long t0 = (long)blockIdx.x * kRopeTokens;
  const int nt = (int)min((long)kRopeTokens, tokens - t0);
  const int n = nt * heads * cpr;
  const bf16* xb = x + t0 * heads * d;
  bf16* yb = y + t0 * heads * d;
  // chunk i: row (token, head) i / cpr of this workgroup, columns 8 (i % cpr)
  auto at = [&](int i) { return (long)(i / cpr) * d + 8 * (i % cpr); };
  bf16x8 lo[kRopeAhead], hi[kRopeAhead];
#pragma unroll
  for (int q = 0; q < kRopeAhead; ++q) {
    const int i = threadIdx.x + q * kRowThreads;
    if (i < n) {
      lo[q] = *(const bf16x8*)(xb + at(i));
      hi[q] = *(const bf16x8*)(xb + at(i) + half);
    }
  }
  for (int i = threadIdx.x; i < nt * half; i += kRowThreads) {
    const int j = i % half;
    const double freq = pow(theta, -2.0 * (double)j / (double)d);
    cs[i / half][j] = rope_angle((double)(pos0 + t0 + i / half), freq, sign);
  }
  __syncthreads();
  auto rotate = [&](int i, const bf16x8& a, const bf16x8& b) {
    const float2* c = &cs[i / cpr / heads][8 * (i % cpr)];
    bf16x8 oa, ob;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      oa[k] = (bf16)((float)a[k] * c[k].x - (float)b[k] * c[k].y);
      ob[k] = (bf16)((float)b[k] * c[k].x + (float)a[k] * c[k].y);
    }
    *(bf16x8*)(yb + at(i)) = oa;
    *(bf16x8*)(yb + at(i) + half) = ob;
  };
#pragma unroll
  for (int q = 0; q < kRopeAhead; ++q) {
    const int i = threadIdx.x + q * kRowThreads;
    if (i < n) rotate(i, lo[q], hi[q]);
  }
  for (int i = threadIdx.x + kRopeAhead * kRowThreads; i < n; i += kRowThreads) {
    const bf16x8 a = *(const bf16x8*)(xb + at(i)), b = *(const bf16x8*)(xb + at(i) + half);
    rotate(i, a, b);
  }
}

// any even head dim: one workgroup per token; thread (head, j) rotates the
// pair (j, j + d/2)
__global__ __launch_bounds__(kRowThreads) void rope_kernel(const bf16* x, bf16* y, int heads, int d, int pos0,
                                                           double theta, float sign) {
  const long t = blockIdx.x;
  const int half = d / 2;
  for (int i = threadIdx.x; i < heads * half; i += kRowThreads) {
    const int h = i / half, j = i % half;
    const float2 c = rope_angle((double)(pos0 + t), pow(theta, -2.0 * (double)j / (double)d), sign);
    const long base = (t * heads + h) * d;
    const float a = (float)x[base + j], b = (float)x[base + j + half];
    y[base + j] = (bf16)(a * c.x - b * c.y);
    y[base + j + half] = (bf16)(b * c.x + a * c.y);
  }
}

__global__ __launch_bounds__(256) void swiglu_fwd_kernel(const bf16* __restrict__ g, const bf16* __restrict__ u,
                                                         bf16* __restrict__ m, long n8) {
  const long i = (long)blockIdx.x * 256 + threadIdx.x;
  if (i >= n8) return;
  float gv[8], uv[8], o[8];
  load8(g + 8 * i, gv);
  load8(u + 8 * i, uv);
#pragma unroll
  for (int j = 0; j < 8; ++j) o[j] = gv[j] / (1.f + __expf(-gv[j])) * uv[j];
  store8(m + 8 * i, o);
}

__global__ __launch_bounds__(256) void swiglu_bwd_kernel(const bf16* __restrict__ g, const bf16* __restrict__ u,
                                                         const bf16* __restrict__ dm, bf16* __restrict__ dg,
                                                         bf16* __restrict__ du, long n8) {
  const long i = (long)blockIdx.x * 256 + threadIdx.x;
  if (i >= n8) return;
  float gv[8], uv[8], dv[8], og[8], ou[8];
  load8(g + 8 * i, gv);
  load8(u + 8 * i, uv);
  load8(dm + 8 * i, dv);
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const float s = 1.f / (1.f + __expf(-gv[j]));
    const float silu = gv[j] * s;
    og[j] = dv[j] * uv[j] * s * (1.f + gv[j] * (1.f - s));
    ou[j] = dv[j] * silu;
  }
  store8(dg + 8 * i, og);
  store8(du + 8 * i, ou);
}

// dst (+)= src, bf16 into fp32: a weight gradient's part added to the sum.
// HBM bound; as separate conversion and addition passes it moves 18 bytes per
// value (and 4 to clear the sum first), here 10, and 6 for the first part.
// Measured on a Llama3-8B layer (218 M weights, five parts): 3.4 ms of the step
// as passes, 1.6 ms here (6.3 TB/s).
template <bool OVERWRITE>
__global__ __launch_bounds__(256) void grad_accumulate_kernel(const bf16* __restrict__ src, float4* __restrict__ dst,
                                                              long n8) {
  const long i = (long)blockIdx.x * 256 + threadIdx.x;
  if (i >= n8) return;
  float v[8];
  load8(src + 8 * i, v);
  float4 a = make_float4(v[0], v[1], v[2], v[3]), b = make_float4(v[4], v[5], v[6], v[7]);
  if constexpr (!OVERWRITE) {
    const float4 c = dst[2 * i], d = dst[2 * i + 1];
    a.x += c.x; a.y += c.y; a.z += c.z; a.w += c.w;
    b.x += d.x; b.y += d.y; b.z += d.z; b.w += d.w;
  }
  dst[2 * i] = a;
  dst[2 * i + 1] = b;
}

hipError_t launch_grad_accumulate(long n, const void* src, float* dst, bool overwrite, hipStream_t st) {
  const long n8 = n / 8;
  if (n8 == 0) return hipSuccess;
  ProfileScope ps("grad_accumulate", st);
  const dim3 grid((unsigned)((n8 + 255) / 256));
  if (overwrite)
    hipLaunchKernelGGL(grad_accumulate_kernel<true>, grid, dim3(256), 0, st, (const bf16*)src, (float4*)dst, n8);
  else
    hipLaunchKernelGGL(grad_accumulate_kernel<false>, grid, dim3(256), 0, st, (const bf16*)src, (float4*)dst, n8);
  return hipGetLastError();
}

hipError_t launch_rmsnorm_fwd(int rows, int width, float eps, const void* x, void* y, float* rstd, hipStream_t st) {
  if (rows == 0) return hipSuccess;
  ProfileScope ps("rmsnorm_fwd", st);
  hipLaunchKernelGGL(rmsnorm_fwd_kernel, dim3(rows), dim3(kRowThreads), 0, st, (const bf16*)x, (bf16*)y, rstd, width,
                     eps);
  return hipGetLastError();
}

hipError_t launch_rmsnorm_bwd(int rows, int width, const void* x, const float* rstd, const void* dy, const void* add,
                              void* dx, hipStream_t st) {
  if (rows == 0) return hipSuccess;
  ProfileScope ps("rmsnorm_bwd", st);
  hipLaunchKernelGGL(rmsnorm_bwd_kernel, dim3(rows), dim3(kRowThreads), 0, st, (const bf16*)x, rstd,
                     (const bf16*)dy, (const bf16*)add, (bf16*)dx, width);
  return hipGetLastError();
}

hipError_t launch_rope(int tokens, int heads, int d, int pos0, double theta, const void* x, void* y, bool inverse,
                       hipStream_t st) {
  if (tokens == 0) return hipSuccess;
  ProfileScope ps(inverse ? "rope_bwd" : "rope_fwd", st);
  const float sign = inverse ? -1.f : 1.f;
  if (d % 16 == 0 && d / 2 <= kRopeMaxHalf)
    hipLaunchKernelGGL(rope_shared_kernel, dim3((tokens - 1) / kRopeTokens + 1), dim3(kRowThreads), 0, st,
                       (const bf16*)x, (bf16*)y, (long)tokens, heads, d, pos0, theta, sign);
  else
    hipLaunchKernelGGL(rope_kernel, dim3(tokens), dim3(kRowThreads), 0, st, (const bf16*)x, (bf16*)y, heads, d, pos0,
                       theta, sign);
  return hipGetLastError();
}

hipError_t launch_swiglu_fwd(long n, const void* g, const void* u, void* m, hipStream_t st) {
  const long n8 = n / 8;
  if (n8 == 0) return hipSuccess;
  ProfileScope ps("swiglu_fwd", st);
  hipLaunchKernelGGL(swiglu_fwd_kernel, dim3((unsigned)((n8 + 255) / 256)), dim3(256), 0, st, (const bf16*)g,
                     (const bf16*)u, (bf16*)m, n8);
  return hipGetLastError();
}

hipError_t launch_swiglu_bwd(long n, const void* g, const void* u, const void* dm, void* dg, void* du,
                             hipStream_t st) {
  const long n8 = n / 8;
  if (n8 == 0) return hipSuccess;
  ProfileScope ps("swiglu_bwd", st);
  hipLaunchKernelGGL(swiglu_bwd_kernel, dim3((unsigned)((n8 + 255) / 256)), dim3(256), 0, st, (const bf16*)g,
                     (const bf16*)u, (const bf16*)dm, (bf16*)dg, (bf16*)du, n8);
  return hipGetLastError();
}

}  // namespace spr
