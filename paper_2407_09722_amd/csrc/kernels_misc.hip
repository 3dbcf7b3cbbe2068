// Row-wise pieces of the decoder pass: embedding gather, RMSNorm (wavefront reductions), the rotary
// table and the row-wise logsumexp of the logits.
// All of them move a few KB..MB per launch; they are latency bound, not bandwidth bound.
#include "common.h"

namespace mtad {

// The inputs of a pass, one workgroup per row: h[row] = E[tok[row]]; bf16 models: also planes of h*g0 (input of the
// first fused RMSNorm) and ssq[row] = sum h^2; and the row's rotary table, table[row][i] = (cos, sin)(pos[row] *
// theta^(-2i/head_dim)), evaluated in double so that positions in the thousands keep float32-exact angles.
template <typename T>
__global__ __launch_bounds__(256) void embed_kernel(const T* __restrict__ E, const int32_t* __restrict__ tok, float* __restrict__ h, int d,
                                                    int vocab, const float* __restrict__ g0, bf16_t* __restrict__ planes,
                                                    float* __restrict__ ssq, const int32_t* __restrict__ pos, float2* __restrict__ table,
                                                    int half, float theta, int ncg) {
  __shared__ float sh[4];
  const int row = blockIdx.x;
  for (int i = threadIdx.x; i < half; i += blockDim.x) {
    const double inv_freq = pow((double)theta, -(double)i / (double)half);
    const double ang = (double)pos[row] * inv_freq;
    double sn, cs;
    sincos(ang, &sn, &cs);
    table[(int64_t)row * half + i] = make_float2((float)cs, (float)sn);
  }
  int t = tok[row];
  if (t < 0 || t >= vocab) t = 0;  // inactive rows carry no meaningful token
  const T* e = E + (int64_t)t * d;
  float ss = 0.f;
  for (int i = threadIdx.x * 4; i < d; i += blockDim.x * 4) {  // d is a multiple of 4 (checked at create)
    float v[4];
    if constexpr (sizeof(T) == 2) {
      const ushort4 b = *(const ushort4*)(e + i);
      v[0] = bf16_to_f32(b.x); v[1] = bf16_to_f32(b.y); v[2] = bf16_to_f32(b.z); v[3] = bf16_to_f32(b.w);
    } else {
      const float4 f = *(const float4*)(e + i);
      v[0] = f.x; v[1] = f.y; v[2] = f.z; v[3] = f.w;
    }
    *(float4*)(h + (int64_t)row * d + i) = make_float4(v[0], v[1], v[2], v[3]);
    if (planes) {
      const float4 g = *(const float4*)(g0 + i);
      ushort4 hi, lo;
      split_bf16(v[0] * g.x, hi.x, lo.x);
      split_bf16(v[1] * g.y, hi.y, lo.y);
      split_bf16(v[2] * g.z, hi.z, lo.z);
      split_bf16(v[3] * g.w, hi.w, lo.w);
      ss += v[0] * v[0];
      ss += v[1] * v[1];
      ss += v[2] * v[2];
      ss += v[3] * v[3];
      *(ushort4*)(planes + act_offset(ncg, (int)gridDim.x, d, 0, row, i)) = hi;
      *(ushort4*)(planes + act_offset(ncg, (int)gridDim.x, d, 1, row, i)) = lo;
    }
  }
  if (planes) {
    ss = block_sum(ss, sh);
    if (threadIdx.x == 0) ssq[row] = ss;
  }
}

hipError_t launch_embed(int dtype, const void* E, const int32_t* tok, float* h, int rows, int d, int vocab, const float* g0,
                        void* planes, float* ssq, const int32_t* pos, float2* table, int head_dim, float theta, int ncg, hipStream_t s) {
  if (rows <= 0) return hipSuccess;
  if (dtype == 1)
    hipLaunchKernelGGL((embed_kernel<bf16_t>), dim3(rows), dim3(256), 0, s, (const bf16_t*)E, tok, h, d, vocab, g0, (bf16_t*)planes, ssq, pos,
                       table, head_dim / 2, theta, ncg);
  else
    hipLaunchKernelGGL((embed_kernel<float>), dim3(rows), dim3(256), 0, s, (const float*)E, tok, h, d, vocab, nullptr, nullptr, nullptr, pos,
                       table, head_dim / 2, theta, 0);
  return hipGetLastError();
}

// out[row][i] = h[row][i] / sqrt(mean(h[row]^2) + eps) * g[i].  No pass runs it (the products normalise their input themselves): it is
// the component entry point mtad_k_rmsnorm.
template <typename T>
__global__ __launch_bounds__(256) void rmsnorm_kernel(const float* __restrict__ h, const float* __restrict__ g, T* __restrict__ out,
                                                      int d, float eps) {
  __shared__ float sh[4];
  const int row = blockIdx.x;
  const int64_t lo_plane = (int64_t)gridDim.x * d;
  const float* x = h + (int64_t)row * d;
  float ss = 0.f;
  for (int i = threadIdx.x * 4; i < d; i += 1024) {
    const float4 v = *(const float4*)(x + i);
    ss += v.x * v.x + v.y * v.y + v.z * v.z + v.w * v.w;
  }
  ss = block_sum(ss, sh);
  const float inv = 1.0f / sqrtf(ss / (float)d + eps);
  for (int i = threadIdx.x * 4; i < d; i += 1024) {
    const float4 v = *(const float4*)(x + i);
    const float4 gg = *(const float4*)(g + i);
    const float o0 = v.x * inv * gg.x, o1 = v.y * inv * gg.y, o2 = v.z * inv * gg.z, o3 = v.w * inv * gg.w;
    if constexpr (sizeof(T) == 2) {
      ushort4 hi, lo;
      split_bf16(o0, hi.x, lo.x);
      split_bf16(o1, hi.y, lo.y);
      split_bf16(o2, hi.z, lo.z);
      split_bf16(o3, hi.w, lo.w);
      *(ushort4*)(out + (int64_t)row * d + i) = hi;
      *(ushort4*)(out + lo_plane + (int64_t)row * d + i) = lo;
    } else {
      *(float4*)(out + (int64_t)row * d + i) = make_float4(o0, o1, o2, o3);
    }
  }
}

hipError_t launch_rmsnorm(int dtype, const float* h, const float* g, void* out, int rows, int d, float eps, hipStream_t s) {
  if (rows <= 0) return hipSuccess;
  if (d % 4) return hipErrorInvalidValue;
  if (dtype == 1) hipLaunchKernelGGL((rmsnorm_kernel<bf16_t>), dim3(rows), dim3(256), 0, s, h, g, (bf16_t*)out, d, eps);
  else hipLaunchKernelGGL((rmsnorm_kernel<float>), dim3(rows), dim3(256), 0, s, h, g, (float*)out, d, eps);
  return hipGetLastError();
}

// lse[row] = log(sum_v exp(logits[row][v])), max-shifted; one block per row
__global__ __launch_bounds__(256) void row_lse_kernel(const float* __restrict__ logits, float* __restrict__ lse, int vocab) {
  __shared__ float sh[4];
  const float* x = logits + (int64_t)blockIdx.x * vocab;
  float m = -INFINITY;
  for (int i = threadIdx.x; i < vocab; i += 256) m = fmaxf(m, x[i]);
  m = block_max(m, sh);
  float sum = 0.f;
  for (int i = threadIdx.x; i < vocab; i += 256) sum += expf(x[i] - m);
  sum = block_sum(sum, sh);
  if (threadIdx.x == 0) lse[blockIdx.x] = m + logf(sum);
}

hipError_t launch_row_lse(const float* logits, float* lse, int rows, int vocab, hipStream_t s) {
  if (rows <= 0) return hipSuccess;
  hipLaunchKernelGGL(row_lse_kernel, dim3(rows), dim3(256), 0, s, logits, lse, vocab);
  return hipGetLastError();
}

// lse[row] = log sum exp over the row from per-strip partials (max, sum exp), merged in strip order
__global__ __launch_bounds__(256) void lse_finish_kernel(const float2* __restrict__ part, float* __restrict__ lse, int NP) {
  __shared__ float sh[4];
  const float l = lse_of_row(part + (int64_t)blockIdx.x * NP, NP, sh);
  if (threadIdx.x == 0) lse[blockIdx.x] = l;
}

// The same, fused with the gather of the tree nodes' conditional log-likelihoods: workgroup (sequence s, row c) writes
// lse[s][c] and, for c > 0, logp_cond[s][c] = logits[s][parent(c)][tok(c)] - lse[s][parent(c)], reducing the
// parent row's partials itself (same code, same order: the value equals the one the parent's workgroup writes).
__global__ __launch_bounds__(256) void lse_gather_kernel(const float2* __restrict__ part, float* __restrict__ lse, int NP,
                                                         const float* __restrict__ logits, int M, int V, const int32_t* __restrict__ parent,
                                                         const int32_t* __restrict__ tok, float* __restrict__ logp_cond) {
  __shared__ float sh[4];
  const int idx = blockIdx.x, s = idx / M, c = idx % M;
  const float own = lse_of_row(part + (int64_t)idx * NP, NP, sh);
  if (threadIdx.x == 0) lse[idx] = own;
  float out = 0.f;
  if (c > 0) {  // uniform over the workgroup
    const int p = parent[idx], t = tok[idx];
    if (p >= 0 && p < M && t >= 0 && t < V) {
      __syncthreads();  // sh is reused
      const float lp = lse_of_row(part + ((int64_t)s * M + p) * NP, NP, sh);
      out = logits[((int64_t)s * M + p) * V + t] - lp;
    }
  }
  if (threadIdx.x == 0) logp_cond[idx] = out;
}

hipError_t launch_lse_gather(const float* lse_part, float* lse, int B, int M, int NP, const float* logits, int V, const int32_t* parent,
                             const int32_t* tok, float* logp_cond, hipStream_t s) {
  if (B * M <= 0) return hipSuccess;
  hipLaunchKernelGGL(lse_gather_kernel, dim3(B * M), dim3(256), 0, s, (const float2*)lse_part, lse, NP, logits, M, V, parent, tok, logp_cond);
  return hipGetLastError();
}

hipError_t launch_lse_finish(const float* lse_part, float* lse, int rows, int NP, hipStream_t s) {
  if (rows <= 0) return hipSuccess;
  hipLaunchKernelGGL(lse_finish_kernel, dim3(rows), dim3(256), 0, s, (const float2*)lse_part, lse, NP);
  return hipGetLastError();
}

// Plain streaming copy of n 16-byte words: the reference point for hardware byte counters (it reads and writes
// exactly 16*n bytes) and for the bandwidth a trivially coalesced kernel reaches.
__global__ __launch_bounds__(256) void copy_kernel(const uint4* __restrict__ src, uint4* __restrict__ dst, int64_t n) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) dst[i] = src[i];
}

hipError_t launch_copy(const void* src, void* dst, int64_t bytes, hipStream_t s) {
  const int64_t n = bytes / 16;
  if (n <= 0) return hipSuccess;
  const int64_t want = (n + 255) / 256;
  const int blocks = (int)(want < 256 * 16 ? want : 256 * 16);
  hipLaunchKernelGGL(copy_kernel, dim3(blocks), dim3(256), 0, s, (const uint4*)src, (uint4*)dst, n);
  return hipGetLastError();
}

}  // namespace mtad
