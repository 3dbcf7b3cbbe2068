// Skinny matrix products Y[R][N] = X[R][K] * W[N][K]^T for the few-row projections, FFN and lm_head of the
// draft and target passes: the weight stream that dominates one target pass.
//
// bf16 path.  Weights are tile-packed (pack_matrix_kernel): the 16x32 tile (nt, kt) of the matrix is 1 KiB
// contiguous, laid out exactly as the A operand of v_mfma_f32_16x16x32_bf16 wants it (lane l holds row l%16,
// k = (l/16)*8 .. +8), and the tiles of one 16-feature strip follow each other along k.  A wave therefore
// fetches every A fragment as one fully coalesced 1 KiB read and a workgroup streams one contiguous strip.
// Activations are the B operand, carried as two bf16 planes (hi + lo): the 16 columns of one MFMA hold the hi
// and lo terms of 8 rows, so a weight tile costs one MFMA per 8 rows.
// One workgroup owns one strip; its waves split the k tiles and add their partial sums in a fixed order
// (deterministic).  The epilogue variants fold the neighbouring element-wise work in:
//   STORE   plain store / accumulate; optional per-strip (max, sum-exp) partials of each row (lm_head)
//   RESID   residual add, then the next RMSNorm's input: planes of h*gain and per-strip sums of squares
//   SWIGLU  strips hold 8 gate + 8 up features: silu(gate)*up written as planes
//   QKV     strips hold features i..i+8 and i+hd/2.. of one head: rotary rotation, q to a buffer, k/v to the cache
// A product whose input is RMS-normalised takes planes of h*gain and multiplies its rows by
// 1/sqrt(mean h^2 + eps) afterwards (the factor is common to the whole row, so it commutes with the product).
//
// fp32 path (the tiny all-float32 workload): one wave per output feature or pair of features, plain FMA.
#include "common.h"
#include "gemm.h"
#include "gemm_device.h"

#include <stdlib.h>

#include <type_traits>

namespace mtad {

// ---- packing ------------------------------------------------------------------------------------------

// original row of packed row (nt*16 + j)
__device__ __forceinline__ int packed_src_row(int kind, int nt, int j, int head_dim, int d_ffn) {
  if (kind == PACK_QKV) {
    const int tph = head_dim / 16, head = nt / tph, u = nt % tph;
    return head * head_dim + (j < 8 ? 8 * u + j : head_dim / 2 + 8 * u + (j - 8));
  }
  if (kind == PACK_GATE_UP) return j < 8 ? 8 * nt + j : d_ffn + 8 * nt + (j - 8);
  return nt * 16 + j;
}

__global__ void pack_matrix_kernel(const bf16_t* __restrict__ src, bf16_t* __restrict__ dst, int N, int K, int kind, int head_dim) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;  // one thread per 8-element lane fragment
  const int KT = K / 32;
  if (idx >= (int64_t)(N / 16) * KT * 64) return;
  const int lane = (int)(idx & 63);
  const int64_t tile = idx >> 6;
  const int kt = (int)(tile % KT), nt = (int)(tile / KT);
  const int row = packed_src_row(kind, nt, lane & 15, head_dim, N / 2);
  const uint4 v = *(const uint4*)(src + (int64_t)row * K + kt * 32 + (lane >> 4) * 8);
  *(uint4*)(dst + idx * 8) = v;
}

hipError_t launch_pack_matrix(const void* src, void* dst, int N, int K, int kind, int head_dim, hipStream_t s) {
  const int64_t n = (int64_t)(N / 16) * (K / 32) * 64;
  hipLaunchKernelGGL(pack_matrix_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, (const bf16_t*)src, (bf16_t*)dst, N, K,
                     kind, head_dim);
  return hipGetLastError();
}

// ---- the product -----------------------------------------------------------------------------------------


// One workgroup = one strip of 16 output features; its GW waves interleave over the k tiles (wave w takes tiles
// w, w + GW, ...) in batches of U tiles, and their partial sums meet in LDS in a fixed order (deterministic).
// Columns of the B operand: c < 8 = hi term of row g*8 + c, c >= 8 = lo term of row g*8 + c - 8, so one MFMA per
// weight tile covers 8 rows (NG = ceil(rows / 8) MFMAs per tile).  Wave g < NG finishes row group g.
// Each wave keeps TWO batches in flight (register sets 0 and 1): when a batch has been consumed its registers take
// the batch two places ahead.  Loads complete in issue order, so a wave that waits for its newest load has waited
// for all of them; the activation fragments of a batch (L2 hits) are therefore issued BEFORE its weight tiles, two
// batches ahead of their use, never between a batch's weight loads and its use.  Workgroups are small (512 threads,
// few registers) so that several are resident per compute unit: while one runs its epilogue or waits for its first
// tiles, the others keep the memory pipe full.
// TAG only names the call site (0 draft pass, 1 target pass, 2 component entry point) in kernel traces.

template <int NG, int EPI, int TAG>
__global__ __launch_bounds__(GW * 64) __attribute__((amdgpu_waves_per_eu((NG <= 1 && EPI != EPI_RESID) ? 6 : 4))) void gemm_bf16_kernel(GemmArgs a) {
  constexpr int U = (NG <= 2) ? 4 : (NG <= 4 ? 2 : 1);  // weight tiles per batch and wave
  __shared__ floatx4 red[GW * NG * 64];
  __shared__ float inv_s[NG * 8];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // wave-uniform by construction: keep it scalar
  const int nt = blockIdx.x;
  const int K = a.K, KT = K >> 5;
  const int R = a.R, row0 = a.row0;
  const int rows_here = min(NG * 8, R - row0);
  const int c = lane & 15, kg = lane >> 4;

  // (wave-uniform base) + (32-bit lane offset): the scalar-base addressing mode, one offset register per stream
  const char* strip = (const char*)a.W + (((size_t)nt * KT) << 10);
  const unsigned voff = (unsigned)lane * 16u;
  const ActAddr xa = act_addr(a, lane);

  constexpr int span = U * GW;
  Frag w[2][U], b[2][U][NG];
  gemm_load_b<NG, U>(b[0], xa.X, xa.xoff, xa.kstride, xa.gstride, KT, wave, rows_here, c);
  gemm_load_w<U>(w[0], strip, KT, wave, voff);
  gemm_load_b<NG, U>(b[1], xa.X, xa.xoff, xa.kstride, xa.gstride, KT, wave + span, rows_here, c);
  gemm_load_w<U>(w[1], strip, KT, wave + span, voff);

  floatx4 acc[NG];
#pragma unroll
  for (int g = 0; g < NG; ++g) acc[g] = floatx4{0.f, 0.f, 0.f, 0.f};
  // RESID: the finishing wave requests its residual values and the next norm's gain now.  Products with this epilogue
  // (o, down) have about one workgroup per compute unit, so nothing else covers that latency after the stream.
  float4 pre_h = float4{0.f, 0.f, 0.f, 0.f}, pre_gn = pre_h;
  if constexpr (EPI == EPI_RESID) {
    const int mrel = wave * 8 + (c & 7);
    if (wave < NG && c < 8 && mrel < rows_here) {
      pre_h = *(const float4*)(a.h + (int64_t)(row0 + mrel) * a.N + nt * 16 + kg * 4);
      pre_gn = *(const float4*)(a.g_next + nt * 16 + kg * 4);
    }
  }

  for (int kt = wave; kt < KT; kt += 2 * span) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int k0 = kt + h * span;
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (k0 + u * GW < KT) {
#pragma unroll
          for (int g = 0; g < NG; ++g) acc[g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[h][u].v, b[h][u][g].v, acc[g], 0, 0, 0);
        }
      if (k0 + 2 * span < KT) {
        gemm_load_b<NG, U>(b[h], xa.X, xa.xoff, xa.kstride, xa.gstride, KT, k0 + 2 * span, rows_here, c);
        gemm_load_w<U>(w[h], strip, KT, k0 + 2 * span, voff);
      }
    }
  }
#pragma unroll
  for (int g = 0; g < NG; ++g) red[(wave * NG + g) * 64 + lane] = acc[g];
  gemm_row_factors<false, (NG > 1 ? NG : 1)>(a, inv_s, rows_here, wave, lane, GW);  // after the stream: its loads are L2 hits by now for most workgroups
  __syncthreads();
  if (wave < NG) gemm_finish_group<NG, EPI, false, GW, EPI == EPI_RESID>(a, nt, wave, red, inv_s, rows_here, lane, pre_h, pre_gn);
}

// The same kernel for S strips per workgroup: the activation fragments of a k tile are loaded once and multiplied with
// the S weight tiles of that k tile, so the L2 -> compute-unit traffic of the fragments per weight byte is 1/S of the
// one-strip kernel's (which spends 12 to 15 % of its time on them at 5 rows: measured by knocking the loads out).
// U tiles per batch and strip, two batches in flight as above; the S strips are reduced and finished at the
// same time by different waves.  Used with S = 3 for 4 to 8 rows (U = 2) and 9 to 24 rows (U = 1).
template <int NG, int EPI, int TAG, int S, int U>
__global__ __launch_bounds__(GW * 64) __attribute__((amdgpu_waves_per_eu((S + NG) * U * 8 + S * NG * 4 > 100 ? 2 : 4))) void gemm_bf16_strips_kernel(GemmArgs a) {
  __shared__ floatx4 red[S * GW * NG * 64];
  __shared__ float inv_s[NG * 8];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int K = a.K, KT = K >> 5, NT = a.N >> 4;
  const int R = a.R, row0 = a.row0;
  const int rows_here = min(NG * 8, R - row0);
  const int c = lane & 15;
  const int nt0 = blockIdx.x * S, ns = min(S, NT - nt0);
  const size_t strip_bytes = (size_t)KT << 10;
  const char* strip0 = (const char*)a.W + (size_t)nt0 * strip_bytes;
  const unsigned voff = (unsigned)lane * 16u;
  const ActAddr xa = act_addr(a, lane);

  constexpr int span = U * GW;
  Frag w[2][U][S], b[2][U][NG];
  auto load_w = [&](Frag (&ws)[U][S], int kt) {
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int s2 = 0; s2 < S; ++s2)
        if (kt + u * GW < KT)  // a strip past the last one reads the last one again: never finished
          ws[u][s2].n = __builtin_nontemporal_load((const uintx4*)(strip0 + (size_t)min(s2, ns - 1) * strip_bytes + ((size_t)(kt + u * GW) << 10) + voff));
  };
  gemm_load_b<NG, U>(b[0], xa.X, xa.xoff, xa.kstride, xa.gstride, KT, wave, rows_here, c);
  load_w(w[0], wave);
  gemm_load_b<NG, U>(b[1], xa.X, xa.xoff, xa.kstride, xa.gstride, KT, wave + span, rows_here, c);
  load_w(w[1], wave + span);

  floatx4 acc[S][NG];
#pragma unroll
  for (int s2 = 0; s2 < S; ++s2)
#pragma unroll
    for (int g = 0; g < NG; ++g) acc[s2][g] = floatx4{0.f, 0.f, 0.f, 0.f};

  for (int kt = wave; kt < KT; kt += 2 * span) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int k0 = kt + h * span;
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (k0 + u * GW < KT) {
#pragma unroll
          for (int s2 = 0; s2 < S; ++s2)
#pragma unroll
            for (int g = 0; g < NG; ++g) acc[s2][g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[h][u][s2].v, b[h][u][g].v, acc[s2][g], 0, 0, 0);
        }
      if (k0 + 2 * span < KT) {
        gemm_load_b<NG, U>(b[h], xa.X, xa.xoff, xa.kstride, xa.gstride, KT, k0 + 2 * span, rows_here, c);
        load_w(w[h], k0 + 2 * span);
      }
    }
  }
  gemm_row_factors<false, (NG > 1 ? NG : 1)>(a, inv_s, rows_here, wave, lane, GW);
  // all strips' sums to LDS at once; wave s2 * NG + g then finishes row group g of strip s2, the strips side by side
  // (one after the other, each epilogue's dependent loads, the rotary table, cache slots and residual rows, added up)
#pragma unroll
  for (int s2 = 0; s2 < S; ++s2)
#pragma unroll
    for (int g = 0; g < NG; ++g) red[((s2 * GW + wave) * NG + g) * 64 + lane] = acc[s2][g];
  __syncthreads();
  for (int item = wave; item < S * NG; item += GW) {  // (a ninth item falls to wave 0 again)
    const int s2 = item / NG, g = item % NG;
    if (s2 < ns) gemm_finish_group<NG, EPI>(a, nt0 + s2, g, red + s2 * GW * NG * 64, inv_s, rows_here, lane);
  }
}

// Several strips per workgroup, for passes of more than 8 rows.  With NG row groups a weight tile needs NG activation
// fragments of its own size from L2; a workgroup that works on S strips at once loads the fragments of a k tile
// once and uses them for S weight tiles, so the L2 -> compute-unit traffic per weight byte drops from 1 + NG to
// 1 + NG/S.  Same wave layout as above with U k tiles per batch and wave; the S strips are reduced and finished one
// after the other through the same LDS buffer.  A product with about one strip per compute unit or fewer would leave
// most units idle at S > 1: its reduction dimension is then also cut into KS ranges (grid.y); every workgroup leaves
// its sums in global memory (device-scope write-through stores) and the one that arrives last for a group of strips
// adds the KS partial sums in range order and runs the epilogues (deterministic, same protocol as the attention splits).  S * NG <= 12 (16 for 48 and 64 rows) bounds the accumulator registers.
// U = 2 for two strips (9 to 24 rows, two ranges): 32 KiB of weights are on their way to a compute unit with one tile a batch, less than HBM's
// latency times its share of the rate.  4096 x 11008 at 17 rows 24.6 -> 23.6 us (3.8 TB/s); four tiles a batch 24.2, four ranges 26.1.
template <int NG, int EPI, int U>
__global__ __launch_bounds__(GW * 64) void gemm_bf16_multi_kernel(GemmArgs a, int S) {
  __shared__ int last_s;
  constexpr int SM = U > 1 ? 2 : NG <= 4 ? 12 / NG : (NG <= 6 ? 3 : 4);  // most strips per workgroup
  __shared__ floatx4 red[GW * NG * 64];
  __shared__ float inv_s[NG * 8];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int K = a.K, KT_all = K >> 5, NT = a.N >> 4;
  const int R = a.R, row0 = a.row0;
  const int rows_here = min(NG * 8, R - row0);
  const int c = lane & 15, kg = lane >> 4;
  const int nt0 = blockIdx.x * S, ns = min(S, NT - nt0);
  // this workgroup's range of k tiles [k_lo, KT)
  const int KS = gridDim.y, ks = blockIdx.y;
  const int per = (KT_all + KS - 1) / KS;
  const int k_lo = ks * per, KT = min(KT_all, k_lo + per);

  const char* strip0 = (const char*)a.W + (((size_t)nt0 * KT_all) << 10);
  const size_t strip_bytes = (size_t)KT_all << 10;
  const unsigned voff = (unsigned)lane * 16u;
  const ActAddr xa = act_addr(a, lane);

  constexpr int span = U * GW;
  Frag w[2][U][SM], b[2][U][NG];
  auto load_w = [&](Frag (&ws)[U][SM], int kt) {
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int s2 = 0; s2 < SM; ++s2)
        if (s2 < ns && kt + u * GW < KT)
          ws[u][s2].n = __builtin_nontemporal_load((const uintx4*)(strip0 + s2 * strip_bytes + ((size_t)(kt + u * GW) << 10) + voff));
  };
  gemm_load_b<NG, U>(b[0], xa.X, xa.xoff, xa.kstride, xa.gstride, KT, k_lo + wave, rows_here, c);
  load_w(w[0], k_lo + wave);
  gemm_load_b<NG, U>(b[1], xa.X, xa.xoff, xa.kstride, xa.gstride, KT, k_lo + wave + span, rows_here, c);
  load_w(w[1], k_lo + wave + span);

  floatx4 acc[SM][NG];
#pragma unroll
  for (int s2 = 0; s2 < SM; ++s2)
#pragma unroll
    for (int g = 0; g < NG; ++g) acc[s2][g] = floatx4{0.f, 0.f, 0.f, 0.f};

  for (int kt = k_lo + wave; kt < KT; kt += 2 * span) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int k0 = kt + h * span;
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (k0 + u * GW < KT) {
#pragma unroll
          for (int s2 = 0; s2 < SM; ++s2)
            if (s2 < ns) {
#pragma unroll
              for (int g = 0; g < NG; ++g) acc[s2][g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[h][u][s2].v, b[h][u][g].v, acc[s2][g], 0, 0, 0);
            }
        }
      if (k0 + 2 * span < KT) {
        gemm_load_b<NG, U>(b[h], xa.X, xa.xoff, xa.kstride, xa.gstride, KT, k0 + 2 * span, rows_here, c);
        load_w(w[h], k0 + 2 * span);
      }
    }
  }
  gemm_row_factors<false, (NG > 1 ? 8 : 1)>(a, inv_s, rows_here, wave, lane, GW);  // after the stream (see the single-strip kernel)
  // partial sums of (group, strip s2, row group g, range ks): 64 lanes x 4 floats
  float* const mypart = a.part ? a.part + ((((size_t)blockIdx.x * SM) * NG) * KS) * 256 : nullptr;
  // The strips are reduced through LDS one after the other; (strip s2, row group g) = item s2 * NG + g goes to wave
  // item % GW, which keeps the sum and runs its epilogue after the last reduction, so that the epilogues of all items
  // (dependent loads of rotary table, cache slots, residual rows) overlap instead of queueing behind NG waves.
  constexpr int HELD = (SM * NG + GW - 1) / GW;
  floatx4 held[HELD];
#pragma unroll
  for (int s2 = 0; s2 < SM; ++s2) {
    if (s2 < ns) {  // uniform over the workgroup
      if (s2 > 0) __syncthreads();  // the previous strip's sums have been read
#pragma unroll
      for (int g = 0; g < NG; ++g) red[(wave * NG + g) * 64 + lane] = acc[s2][g];
      __syncthreads();
#pragma unroll
      for (int g = 0; g < NG; ++g) {
        const int item = s2 * NG + g;
        if (wave == item % GW) {
          const floatx4 sum = gemm_sum_waves<NG>(g, red, lane);
          if (KS == 1) {
            held[item / GW] = sum;
          } else {
            float* p = mypart + ((((size_t)s2 * NG + g) * KS + ks) * 64 + lane) * 4;
            st8<true>(p, make_uint2(__float_as_uint(sum[0]), __float_as_uint(sum[1])));
            st8<true>(p + 2, make_uint2(__float_as_uint(sum[2]), __float_as_uint(sum[3])));
          }
        }
      }
    }
  }
  if (KS == 1) {
#pragma unroll
    for (int h = 0; h < HELD; ++h) {
      const int item = h * GW + wave, s2 = item / NG, g = item % NG;
      if (item < SM * NG && s2 < ns) gemm_finish_sum<EPI>(a, nt0 + s2, g, held[h], inv_s, rows_here, lane);
    }
    return;
  }
  // the workgroup that arrives last for this group of strips adds the ranges in order and finishes
  __builtin_amdgcn_s_waitcnt(0);  // the stores have been acknowledged
  __syncthreads();
  if (threadIdx.x == 0) {
    const int prev = __hip_atomic_fetch_add(a.counters + blockIdx.x, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    last_s = (prev == KS - 1);
    if (last_s) __hip_atomic_store(a.counters + blockIdx.x, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);  // clean for the next launch
  }
  __syncthreads();
  if (!last_s) return;
  // (strip s2, row group g) = item s2 * NG + g goes to wave item % GW, as above: all waves share the merges
  for (int item = wave; item < ns * NG; item += GW) {
    const int s2 = item / NG, g = item % NG;
    const float* p = mypart + ((((size_t)s2 * NG + g) * KS) * 64 + lane) * 4;
    floatx4 sum = floatx4{0.f, 0.f, 0.f, 0.f};
    for (int k2 = 0; k2 < KS; ++k2) {
      const uint4 v = ld16<true>(p + (size_t)k2 * 256);
      sum[0] += __uint_as_float(v.x); sum[1] += __uint_as_float(v.y); sum[2] += __uint_as_float(v.z); sum[3] += __uint_as_float(v.w);
    }
    gemm_finish_sum<EPI>(a, nt0 + s2, g, sum, inv_s, rows_here, lane);
  }
}

// Sums of RB values over the wave, row_of_lane(lane) in each lane: the first exchanges halve the number of values instead of
// repeating each of them in both halves (the additions and their order are wave_sum's): 14 additions instead of 48 for RB = 8.
template <int RB>
__device__ __forceinline__ int row_of_lane(int lane) {
  return RB == 8 ? 2 * (lane >> 4) + (lane & 1) : RB == 4 ? lane >> 4 : 0;
}
template <int RB>
__device__ __forceinline__ float wave_sums(const float (&v)[RB], int lane) {
  static_assert(RB == 1 || RB == 4 || RB == 8, "");
  if constexpr (RB == 1) {
    return wave_sum(v[0]);
  } else {
    float c[RB / 2], d[RB / 4];
#pragma unroll
    for (int j = 0; j < RB / 2; ++j) {
      const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[j]), __float_as_uint(v[j + RB / 2]), false, false);
      c[j] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    }
#pragma unroll
    for (int j = 0; j < RB / 4; ++j) {
      const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(c[j]), __float_as_uint(c[j + RB / 4]), false, false);
      float t = __uint_as_float(r[0]) + __uint_as_float(r[1]);
      t += row_turn<8>(t);
      t += row_turn<4>(t);
      t += row_turn<2>(t);
      t += row_turn<1>(t);
      d[j] = t;
    }
    if constexpr (RB == 8) return lane & 1 ? d[1] : d[0];
    return d[0];
  }
}
// float32 models: one wave per output feature, or per pair of features that an element-wise step joins (rotary partners, gate and
// up), RB rows at a time; plain FMA, sums over the wave.  These models are tiny and every kernel of a pass costs its launch:
// normalisation (the row factor commutes with the product, as above), rotation with the cache write and the gating ride on
// the products, five kernels a layer instead of nine (4 layers, d 256, 5 rows: 123 us a pass, 200 before).  What the epilogue reads
// (rotary values, cache slot, the value to add to) is requested ahead of the products and the page while the sums run; with
// wave_sums this took 98.6 instead of 105 us of that pass, 354 instead of 412 of a 256-row prompt (d 256, 4 layers).
// Weights of less than 8 MB: the launch is one memory latency, the loads of RB rows go out together and those past the end are the
// last one again.  From there on what is computed for rows that do not exist costs its share: 8192 x 4096, one row 35.9 us with RB =
// 8, 21.6 with RB = 1 (6.2 TB/s); three rows 35.8, 25.6 with RB = 4; nine rows (8 and 1) 72.9, 57.7 without them.
// REST: the kernel that computes a remainder's rows alone.
template <int RB, int EPI, bool REST>
__global__ __launch_bounds__(256) void gemm_f32_kernel(GemmF32Args a) {
  constexpr bool PAIR = EPI == EPI_SWIGLU || EPI == EPI_QKV;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int item = blockIdx.x * 4 + wave, r0 = blockIdx.y * RB, K = a.K;
  if (item >= (PAIR ? a.N / 2 : a.N)) return;
  int n = item, n2 = item, head = 0, i = 0;  // features; QKV: rotary pair i of a head
  if constexpr (EPI == EPI_SWIGLU) n2 = item + a.N / 2;
  if constexpr (EPI == EPI_QKV) {
    const int half = a.kv.head_dim >> 1;
    head = item / half;
    i = item % half;
    n = head * a.kv.head_dim + i;
    n2 = n + half;
  }
  float acc[RB], acc2[RB], ss[RB];
#pragma unroll
  for (int r = 0; r < RB; ++r) acc[r] = acc2[r] = ss[r] = 0.f;
  const float *w1 = a.W + (int64_t)n * K, *w2 = a.W + (int64_t)n2 * K;
  const int rows = min(RB, a.R - r0);
  // the lane that ends with the sums of a row requests what its epilogue reads ahead of the products
  const int row = row_of_lane<RB>(lane), m = r0 + min(row, rows - 1);
  const bool ends = (lane & 15) < (RB == 8 ? 2 : 1) && (RB > 1 || lane == 0) && row < rows;
  float before = 0.f;
  float2 cs = make_float2(1.f, 0.f);
  int slot = -1;
  if (ends) {
    if constexpr (EPI == EPI_STORE) {
      if (a.accumulate) before = a.Y[(int64_t)m * a.ldy + n];
    }
    if constexpr (EPI == EPI_QKV) {
      if (head < a.n_heads + a.kv.n_kv_heads) cs = a.rope[(int64_t)m * (a.kv.head_dim >> 1) + i];
      if (head >= a.n_heads) slot = a.slot[m];
    }
  }
  auto products = [&](auto ALL, auto GAIN) {  // ALL: RB rows (past the end the last one again), else those there are
#pragma unroll 2
    for (int k = lane * 4; k < K; k += 256) {
      const float4 w = *(const float4*)(w1 + k);
      float4 v = w, g = make_float4(1.f, 1.f, 1.f, 1.f), x[RB];
      if constexpr (PAIR) v = *(const float4*)(w2 + k);
      if constexpr (GAIN) g = *(const float4*)(a.gain + k);
#pragma unroll
      for (int r = 0; r < RB; ++r)
        if (ALL || r < rows) x[r] = *(const float4*)(a.X + (int64_t)(r0 + (ALL ? min(r, rows - 1) : r)) * K + k);
#pragma unroll
      for (int r = 0; r < RB; ++r) {
        if (!ALL && r >= rows) continue;
        if constexpr (GAIN) {
          ss[r] = fmaf(x[r].x, x[r].x, ss[r]);
          ss[r] = fmaf(x[r].y, x[r].y, ss[r]);
          ss[r] = fmaf(x[r].z, x[r].z, ss[r]);
          ss[r] = fmaf(x[r].w, x[r].w, ss[r]);
          x[r].x *= g.x; x[r].y *= g.y; x[r].z *= g.z; x[r].w *= g.w;
        }
        acc[r] = fmaf(w.x, x[r].x, acc[r]);
        acc[r] = fmaf(w.y, x[r].y, acc[r]);
        acc[r] = fmaf(w.z, x[r].z, acc[r]);
        acc[r] = fmaf(w.w, x[r].w, acc[r]);
        if constexpr (PAIR) {
          acc2[r] = fmaf(v.x, x[r].x, acc2[r]);
          acc2[r] = fmaf(v.y, x[r].y, acc2[r]);
          acc2[r] = fmaf(v.z, x[r].z, acc2[r]);
          acc2[r] = fmaf(v.w, x[r].w, acc2[r]);
        }
      }
    }
  };
  constexpr std::true_type YES{};
  constexpr std::false_type NO{};
  const bool whole = !REST || rows == RB || (K < 1024 && rows > RB / 2);  // (a short reduction is all latency, too)
  if (whole) {
    if (a.gain) products(YES, YES);
    else products(YES, NO);
  } else if constexpr (REST) {
    if (a.gain) products(NO, YES);
    else products(NO, NO);
  }
  int64_t token = 0;
  if constexpr (EPI == EPI_QKV) {
    if (slot >= 0 && slot < kv_capacity(a.kv)) token = kv_token_offset(a.kv, m / a.Rseq, slot);
  }
  // (all rows' epilogues side by side)
  float y = wave_sums(acc, lane), y2 = 0.f, q = 0.f;
  if constexpr (PAIR) y2 = wave_sums(acc2, lane);
  if (a.gain) q = wave_sums(ss, lane);
  if (!ends) return;
  if (a.gain) {
    const float inv = 1.0f / sqrtf(q / (float)K + a.eps);
    y *= inv;
    y2 *= inv;
  }
  if constexpr (EPI == EPI_SWIGLU) {
    a.Y[(int64_t)m * a.ldy + item] = y / (1.0f + expf(-y)) * y2;
  } else if constexpr (EPI == EPI_QKV) {
    const int hd = a.kv.head_dim, KVH = a.kv.n_kv_heads, H = a.n_heads;
    if (head < H + KVH) {  // q and k heads are rotated
      const float t = fmaf(y, cs.x, -(y2 * cs.y));
      y2 = fmaf(y2, cs.x, y * cs.y);
      y = t;
    }
    if (head < H) {
      a.Y[(int64_t)m * a.ldy + n] = y;
      a.Y[(int64_t)m * a.ldy + n2] = y2;
      return;
    }
    if (slot < 0) return;
    if (slot >= kv_capacity(a.kv)) {
      atomicOr(a.status, (uint32_t)ST_KV_CAP);
      return;
    }
    const bool is_k = head < H + KVH;
    float* const dst = (float*)(is_k ? a.kv.k : a.kv.v) + (int64_t)a.layer * a.kv.layer_stride + token +
                       (int64_t)(head - (is_k ? H : H + KVH)) * hd + i;
    dst[0] = y;
    dst[hd >> 1] = y2;
  } else {
    a.Y[(int64_t)m * a.ldy + n] = a.accumulate ? before + y : y;
  }
}

template <int RB, bool REST>
static hipError_t run_f32(const GemmF32Args& a, int epi, hipStream_t s) {
  const int items = (epi == EPI_SWIGLU || epi == EPI_QKV) ? a.N / 2 : a.N;
  const dim3 grid((items + 3) / 4, (a.R + RB - 1) / RB), block(256);
  switch (epi) {
    case EPI_STORE: hipLaunchKernelGGL((gemm_f32_kernel<RB, EPI_STORE, REST>), grid, block, 0, s, a); break;
    case EPI_SWIGLU: hipLaunchKernelGGL((gemm_f32_kernel<RB, EPI_SWIGLU, REST>), grid, block, 0, s, a); break;
    case EPI_QKV: hipLaunchKernelGGL((gemm_f32_kernel<RB, EPI_QKV, REST>), grid, block, 0, s, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_gemm_f32(const GemmF32Args& a, int epi, hipStream_t s) {
  if (a.R <= 0) return hipSuccess;
  if (a.K % 4) return hipErrorInvalidValue;
  if ((int64_t)a.N * a.K < (2 << 20)) return run_f32<8, false>(a, epi, s);
  if (a.R == 1) return run_f32<1, false>(a, epi, s);
  return a.R <= 4 ? run_f32<4, true>(a, epi, s) : run_f32<8, true>(a, epi, s);
}

template <int NG, int EPI, int TAG>
static hipError_t run_one(const GemmArgs& a, hipStream_t s) {
  hipLaunchKernelGGL((gemm_bf16_kernel<NG, EPI, TAG>), dim3(a.N / 16), dim3(GW * 64), 0, s, a);
  return hipGetLastError();
}

template <int NG, int EPI>
static hipError_t run_tag(const GemmArgs& a, int tag, hipStream_t s) {
  if constexpr (NG <= 3) {
    if (tag == 1) return run_one<NG, EPI, 1>(a, s);
    if (tag == 2) return run_one<NG, EPI, 2>(a, s);
  }
  return run_one<NG, EPI, 0>(a, s);
}

template <int NG, int EPI, int S, int U>
static hipError_t run_strips(const GemmArgs& a, int tag, hipStream_t s) {
  const int NT = a.N / 16;
  const dim3 grid((NT + S - 1) / S), block(GW * 64);
  if (tag == 1) hipLaunchKernelGGL((gemm_bf16_strips_kernel<NG, EPI, 1, S, U>), grid, block, 0, s, a);
  else if (tag == 2) hipLaunchKernelGGL((gemm_bf16_strips_kernel<NG, EPI, 2, S, U>), grid, block, 0, s, a);
  else hipLaunchKernelGGL((gemm_bf16_strips_kernel<NG, EPI, 0, S, U>), grid, block, 0, s, a);
  return hipGetLastError();
}

template <int NG, int EPI, int U = 1>
static hipError_t run_multi(const GemmArgs& a, int S, int KS, hipStream_t s) {
  const int NT = a.N / 16;
  hipLaunchKernelGGL((gemm_bf16_multi_kernel<NG, EPI, U>), dim3((NT + S - 1) / S, KS), dim3(GW * 64), 0, s, a, S);
  return hipGetLastError();
}

static int device_cus() {
  static const int n_cus = [] {
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) cus = 0;
    return cus > 0 ? cus : 256;
  }();
  return n_cus;
}

// Products with at most SPLIT_MAX_STRIPS strips (about one per compute unit) take 4 strips per workgroup and cut the
// reduction dimension 4 ways when a workspace is offered; the workspace is sized for that.
constexpr int SPLIT_MAX_STRIPS = 384, SPLIT_S = 4, SPLIT_KS = 4, SPLIT_NG_MAX = 8;
size_t gemm_split_floats(int N) {
  const int NT = N / 16;
  return NT > SPLIT_MAX_STRIPS ? 0 : (size_t)((NT + SPLIT_S - 1) / SPLIT_S) * SPLIT_S * SPLIT_NG_MAX * SPLIT_KS * 256;
}
int gemm_split_counters(int N) {
  return N / 16 > SPLIT_MAX_STRIPS ? 0 : (N / 16 + 1) / 2;  // groups of at least 2 strips
}

// Strips per workgroup for a product with NT strips and NG row groups.  Cost model (fits the measured times at 17, 41
// and 64 rows): the busiest compute unit works on rounds * S strips, and a strip costs in proportion to the bytes
// that reach the compute unit per weight byte, 1 + NG/S; so minimise rounds * (S + NG), larger S on ties.
static int strips_per_group(int NT, int NG) {
  const int n_cus = device_cus();
  if (NG < 2) return 1;
  const int smax = NG <= 4 ? 12 / NG : (NG <= 6 ? 3 : 4);
  int best = 1, best_cost = 0x7fffffff;
  for (int S = 1; S <= smax; ++S) {
    const int groups = (NT + S - 1) / S;
    const int cost = ((groups + n_cus - 1) / n_cus) * (S + NG);
    if (cost <= best_cost) {
      best = S;
      best_cost = cost;
    }
  }
  return best;
}

template <int EPI>
static hipError_t run_epi(GemmArgs a, int tag, hipStream_t s) {
  // at most 64 rows per launch (8 row groups); more rows re-stream the weights per 64-row slab
  for (int r0 = 0; r0 < a.R; r0 += 64) {
    a.row0 = r0;
    const int ng = ((a.R - r0 < 64 ? a.R - r0 : 64) + 7) / 8;
    hipError_t e;
    const int ngt = ng <= 4 ? ng : (ng <= 6 ? 6 : 8);
    int S = strips_per_group(a.N / 16, ngt), KS = 1;
    const int smax = ngt <= 4 ? 12 / ngt : (ngt <= 6 ? 3 : 4);
    // worth its exchange when every wave keeps at least 8 k tiles, or with 64 rows (measured at 17, 41 and 64 rows)
    if (ng >= 2 && a.part && a.counters && a.N / 16 <= SPLIT_MAX_STRIPS && ((a.K >> 5) >= SPLIT_KS * GW * 8 || (ng >= 7 && (a.K >> 5) >= SPLIT_KS * GW * 2))) {
      S = smax < SPLIT_S ? smax : SPLIT_S;  // share the fragments between strips, keep every compute unit busy by cutting k
      KS = SPLIT_KS;
      if (ng <= 3) S = KS = 2;  // 9 to 24 rows: two strips and two ranges (C4 verify 4.12 -> 4.05 ms; 3 x 2, 4 x 2, 2 x 3 and 2 x 4
                                // slower; the same cut for the o projection, 128 k tiles, slower too)
      // the exchange must fit what the caller offers ((group, strip slot, row group, range) x 256 floats, a counter per group)
      const int groups = (a.N / 16 + S - 1) / S;
      if ((size_t)groups * smax * ngt * KS * 256 > a.part_floats || groups > a.counters_n) {
        S = strips_per_group(a.N / 16, ngt);
        KS = 1;
      }
    }
    // 9 to 24 rows, no k split, at least two strips per compute unit: the three-strip kernel with two or three row
    // groups, whose epilogues run side by side (C3 target at 9 and 12 rows: 3.47 -> 3.39 ms per pass; C4, 17 rows:
    // 4.22 -> 4.12 ms)
    if (KS == 1 && (ng == 2 || ng == 3) && a.N / 16 >= 2 * device_cus()) {
      e = ng == 2 ? run_strips<2, EPI, 3, 1>(a, tag, s) : run_strips<3, EPI, 3, 1>(a, tag, s);
      if (e != hipSuccess) return e;
      continue;
    }
    if (S > 1) {
      if (KS == 2) e = ng <= 2 ? run_multi<2, EPI, 2>(a, S, KS, s) : run_multi<3, EPI, 2>(a, S, KS, s);  // (two strips: registers for two tiles a batch)
      else if (ng <= 2) e = run_multi<2, EPI>(a, S, KS, s);
      else if (ng <= 3) e = run_multi<3, EPI>(a, S, KS, s);
      else if (ng <= 4) e = run_multi<4, EPI>(a, S, KS, s);
      else if (ng <= 6) e = run_multi<6, EPI>(a, S, KS, s);
      else e = run_multi<8, EPI>(a, S, KS, s);
      if (e != hipSuccess) return e;
      continue;
    }
    // 4 to 8 rows and at least two strips per compute unit: three strips per workgroup share the activation fragments
    // (measured on the 7B-shaped QKV, gate/up and lm_head products: 6, 10 and 4 % faster at 5 rows, 17, 19 and 15 % at 8;
    // slower at 1 row; two, four, five or six strips per workgroup all slower than three; no gain at 9 to 24 rows over
    // the kernel below that already shares fragments there)
    if (ng <= 1 && a.R - r0 >= 4 && a.N / 16 >= 2 * device_cus()) e = run_strips<1, EPI, 3, 2>(a, tag, s);
    else if (ng <= 1) e = run_tag<1, EPI>(a, tag, s);
    else if (ng <= 2) e = run_tag<2, EPI>(a, tag, s);
    else if (ng <= 3) e = run_tag<3, EPI>(a, tag, s);
    else if (ng <= 4) e = run_tag<4, EPI>(a, tag, s);
    else if (ng <= 6) e = run_tag<6, EPI>(a, tag, s);
    else e = run_tag<8, EPI>(a, tag, s);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// Passes of many rows take both operands through LDS (kernels_gemm_dma.hip): from 65 rows up always (840 shapes of 1024 to 32000
// features and 256 to 13824 terms), from 25 rows up where the output gives half of the compute units a workgroup of 8 strips, and for
// narrower outputs where the reduction is long enough to be cut: from how many terms on depends on the rows, and on how even the
// strips come out over the compute units in the kernels above.  us, above / there, on both sides of the lines:
//   strips    rows     below the line               from the line on
//   64        25       4096: 10.5 / 9.6             5120: 12.6 / 10.5
//             40       3072: 9.6 / 9.7              4096: 12.1 / 10.0
//             64       2048: 9.2 / 9.9              3072: 12.7 / 10.5
//   256       32       5120: 15.0 / 16.0            8192: 22.8 / 22.7
//             40       4096: 14.1 / 15.5            5120: 17.2 / 16.9
//             64       3072: 14.3 / 15.0            4096: 18.6 / 16.5
//   384       32       4096: 16.4 / 17.3            5120: 19.8 / 19.5
//   512       32       8192: 31.2 / 34.1            11008: 42.0 / 41.0
//   640       40       5120: 27.4 / 27.2 to 31      5632: 29.7 / 28.7
//   768       48       5120: 30.5 / 32.4            8192: 46.4 / 45.5
// One line for all of them (4096 terms from 40 rows on, 5120 below, none from 57) costs up to two thirds of a call: 1024 x 1024 at
// 64 rows 9.6 us instead of 5.8, 12288 x 5120 at 25 rows 29.8 instead of 25.9.
constexpr int NEVER = 0x7fffffff;
static int dma_min_terms(int R, int NT) {
  const int rows = R < 33 ? 0 : R < 40 ? 1 : R < 49 ? 2 : R < 57 ? 3 : 4, cus = device_cus();
  const bool even = NT * 20 >= (NT + cus - 1) / cus * cus * 19;  // all compute units have the same count of strips, nearly
  typedef int Terms[5];
  constexpr Terms even_narrow{8192, 5120, 5120, 4096, 4096}, narrow{5120, 5120, 4096, 4096, 3072}, two_rounds{10240, 5120, 5120, 5120, 5120},
      more{8192, 5632, 5632, 5120, 5120}, three_rounds{NEVER, 10240, 8192, 5120, 5120}, rest{5120, 5120, 5120, 5120, 5120};
  if (NT <= SPLIT_MAX_STRIPS) return even ? even_narrow[rows] : narrow[rows];
  if (NT <= 2 * cus) return even ? two_rounds[rows] : rest[rows];
  if (NT <= 5 * cus / 2) return more[rows];
  return NT <= 3 * cus ? three_rounds[rows] : rest[rows];
}

static bool use_dma(const GemmArgs& a) {
  if (!a.ncg && (!a.xfrag || a.xfrag_elems < gemm_dma_xfrag_elems(a.R, a.K))) return false;  // needs fragment order or its scratch
  if (a.R >= 65) return true;
  if (a.R < 25) return false;
  return gemm_dma_wide(a.N) || (a.part && a.K >= dma_min_terms(a.R, a.N >> 4));
}

hipError_t launch_gemm_bf16(const GemmArgs& a, int epi, int tag, hipStream_t s, int* np) {
  if (np) *np = a.N >> 4;
  if (a.R <= 0) return hipSuccess;
  if ((a.N % 16) || (a.K % 32)) return hipErrorInvalidValue;
  if (use_dma(a) && (epi != EPI_STORE || (a.ldy % 4) == 0)) return launch_gemm_bf16_dma(a, epi, s, np);
  if (a.R > 256) return hipErrorInvalidValue;
  switch (epi) {
    case EPI_STORE: return (a.ldy % 4) ? hipErrorInvalidValue : run_epi<EPI_STORE>(a, tag, s);
    case EPI_RESID: return run_epi<EPI_RESID>(a, tag, s);
    case EPI_SWIGLU: return run_epi<EPI_SWIGLU>(a, tag, s);
    case EPI_QKV: return run_epi<EPI_QKV>(a, tag, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace mtad

// For the tests: whether a product of bfloat16 weights goes to the many-row kernel.
extern "C" int mtad_test_gemm_many_rows(const void* args, size_t bytes) {
  return args && bytes == sizeof(mtad::GemmArgs) ? mtad::use_dma(*(const mtad::GemmArgs*)args) : -1;
}
