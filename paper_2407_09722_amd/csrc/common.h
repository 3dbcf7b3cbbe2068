// Internal declarations shared by the kernel files and the C-ABI layer of libmtad.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mtad {

typedef uint16_t bf16_t;  // bfloat16 bit pattern
typedef _Float16 kv16_t;  // storage type of the KV cache of a bfloat16 model: IEEE half (3 more mantissa bits at the same size)

__device__ __forceinline__ float bf16_to_f32(bf16_t b) { return __uint_as_float(((uint32_t)b) << 16); }

// float32 -> bfloat16, round to nearest even: the conversion instruction of gfx950, which gives the same bits as adding
// 0x7FFF + (bit 16) to the pattern for every float32 that is not a NaN (checked over all of them) in a fifth of the instructions
__device__ __forceinline__ bf16_t f32_to_bf16(float f) {
  const __bf16 h = (__bf16)f;
  bf16_t b;
  __builtin_memcpy(&b, &h, 2);
  return b;
}
__device__ __forceinline__ float round_bf16(float f) { return bf16_to_f32(f32_to_bf16(f)); }
// Two-term bfloat16 split of a float32 activation: x ~= hi + lo with a relative error of about 2^-17.
// Matrix-product inputs are carried this way so that their rounding stays far below the weights' own.
__device__ __forceinline__ void split_bf16(float x, bf16_t& hi, bf16_t& lo) {
  hi = f32_to_bf16(x);
  lo = f32_to_bf16(x - bf16_to_f32(hi));
}

// The same for four values, as they are stored.
__device__ __forceinline__ void split_bf16_x4(const float (&x)[4], uint2& hi, uint2& lo) {
  typedef float f4 __attribute__((ext_vector_type(4)));
  typedef __bf16 b4 __attribute__((ext_vector_type(4)));
  const f4 v = {x[0], x[1], x[2], x[3]};
  const b4 h = __builtin_convertvector(v, b4), l = __builtin_convertvector(v - __builtin_convertvector(h, f4), b4);
  __builtin_memcpy(&hi, &h, 8);
  __builtin_memcpy(&lo, &l, 8);
}

// Element offset of activation (plane, row, feature k) of a pass of R rows and K features.  ncg == 0: two planes
// [2][R][K].  ncg > 0 (= ceil(R / 8)): operand-fragment order, the B operand of v_mfma_f32_16x16x32_bf16 for 8 rows at a
// time, where lane (k%32)/8 * 16 + plane * 8 + row % 8 holds 8 consecutive features of fragment (k / 32, row / 8):
//   R > 24   [K/32][ncg][64 lanes][8]: whole fragments, the slots of rows past R unused (the many-row kernel copies
//            them to LDS line by line);
//   R <= 24  [K/32][4 k groups][2 planes][R rows][8]: the same order with the unused row slots left out: a k tile's
//            fragments are 128 R contiguous bytes (5 cache lines at 5 rows instead of 8, 17 at 17 rows instead of 24);
//            row group g of a (k group, plane) block starts 128 g bytes into it.
// Products read this order (whole cache lines per fragment instead of 64-byte pieces of 16 rows); whatever produces
// their input writes it.
constexpr int ACT_COMPACT_ROWS = 24;  // passes of up to this many rows leave the unused row slots out
__host__ __device__ __forceinline__ int64_t act_offset(int ncg, int R, int K, int plane, int row, int k) {
  if (ncg == 0) return ((int64_t)plane * R + row) * K + k;
  if (R <= ACT_COMPACT_ROWS) return ((((int64_t)(k >> 5) * 4 + ((k >> 3) & 3)) * 2 + plane) * R + row) * 8 + (k & 7);
  return ((((int64_t)(k >> 5) * ncg + (row >> 3)) * 64 + ((k >> 3) & 3) * 16 + plane * 8 + (row & 7)) << 3) + (k & 7);
}

// Exchanges between lanes in the vector ALU (swaps of rows of 16 lanes and of halves, rotations inside a row): about a dozen
// clocks each, where a shuffle goes through LDS and takes over a hundred.
template <int N>  // the value N lanes before, around a row of 16 lanes (8: the lane 8 away)
__device__ __forceinline__ float row_turn(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x120 + N, 0xf, 0xf, true));
}
__device__ __forceinline__ float lane_xor16(float v) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);  // even rows; odd rows
  return __uint_as_float(((threadIdx.x >> 4) & 1) ? r[0] : r[1]);
}
__device__ __forceinline__ float lane_xor32(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);  // lower half; upper half
  return __uint_as_float(((threadIdx.x >> 5) & 1) ? r[0] : r[1]);
}
// sum and maximum over the wave, in every lane: the pairs of a butterfly over lane distances 32, 16, 8, 4, 2, 1 (from distance
// 4 on the values repeat with that period, so that a rotation brings the partner's)
__device__ __forceinline__ float wave_sum(float v) {
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  v += row_turn<8>(v);
  v += row_turn<4>(v);
  v += row_turn<2>(v);
  v += row_turn<1>(v);
  return v;
}
__device__ __forceinline__ float wave_max(float v) {
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
  r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
  v = fmaxf(v, row_turn<8>(v));
  v = fmaxf(v, row_turn<4>(v));
  v = fmaxf(v, row_turn<2>(v));
  v = fmaxf(v, row_turn<1>(v));
  return v;
}
// over a workgroup of at most 16 waves, in every thread (waves added in order); sh: one float per wave, free again after the next barrier
__device__ __forceinline__ float block_sum(float v, float* sh) {
  v = wave_sum(v);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  float t = sh[0];
  for (int w = 1; w < (int)(blockDim.x >> 6); ++w) t += sh[w];
  return t;
}
__device__ __forceinline__ float block_max(float v, float* sh) {
  v = wave_max(v);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  float t = sh[0];
  for (int w = 1; w < (int)(blockDim.x >> 6); ++w) t = fmaxf(t, sh[w]);
  return t;
}
// log sum exp of a logits row from the (max, sum exp) partials of its NP strips, by a workgroup of 256 threads.  Rows of up to
// 32768 logits are held in registers between the two reductions, their loads in flight together.
__device__ __forceinline__ float lse_of_row(const float2* __restrict__ p, int NP, float* sh) {
  constexpr int U = 8;
  const int t = threadIdx.x;
  float m = -INFINITY, sum = 0.f;
  if (NP <= 256 * U) {
    float2 v[U];
#pragma unroll
    for (int j = 0; j < U; ++j) v[j] = p[min(t + 256 * j, NP - 1)];
#pragma unroll
    for (int j = 0; j < U; ++j)
      if (t + 256 * j < NP) m = fmaxf(m, v[j].x);
    m = block_max(m, sh);
#pragma unroll
    for (int j = 0; j < U; ++j)
      if (t + 256 * j < NP) sum += v[j].y * expf(v[j].x - m);
  } else {
    for (int i = t; i < NP; i += 256) m = fmaxf(m, p[i].x);
    m = block_max(m, sh);
    for (int i = t; i < NP; i += 256) sum += p[i].y * expf(p[i].x - m);
  }
  sum = block_sum(sum, sh);
  return m + logf(sum);
}

// Device-scope ("coherent") accesses for data that workgroups of ONE kernel hand to each other.  The XCDs' L2
// caches are not coherent with each other; relaxed device-scope atomics compile to write-through stores and
// cache-bypassing loads, which avoids flushing or invalidating whole caches.  COH = false: plain accesses (data
// produced by an earlier kernel).
template <bool COH>
__device__ __forceinline__ uint4 ld16(const void* p) {
  if constexpr (COH) {
    const unsigned long long* q = (const unsigned long long*)p;
    const unsigned long long a = __hip_atomic_load(q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const unsigned long long b = __hip_atomic_load(q + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return make_uint4((uint32_t)a, (uint32_t)(a >> 32), (uint32_t)b, (uint32_t)(b >> 32));
  } else {
    return *(const uint4*)p;
  }
}
template <bool COH>
__device__ __forceinline__ float ld4(const float* p) {
  if constexpr (COH) return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  else return *p;
}
template <bool COH>
__device__ __forceinline__ void st8(void* p, uint2 v) {
  if constexpr (COH)
    __hip_atomic_store((unsigned long long*)p, (unsigned long long)v.x | ((unsigned long long)v.y << 32), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
  else
    *(uint2*)p = v;
}
template <bool COH>
__device__ __forceinline__ void st4(float* p, float v) {
  if constexpr (COH) __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  else *p = v;
}

// Device status bits (sticky, OR-ed by kernels that refuse an out-of-range access)
enum : uint32_t { ST_KV_CAP = 1u, ST_SPEC_WINDOW = 2u, ST_BAD_CATCHUP = 4u, ST_TIMEOUT = 8u };

// Paged KV addressing: element offset of (layer, logical position pos, kv head 0, dim 0)
struct KvView {
  void* k;
  void* v;
  const int32_t* page_table;  // [B][max_pages]
  int32_t* len;               // [B]
  int32_t page_size, max_pages, n_pages;
  int32_t n_kv_heads, head_dim;
  int64_t layer_stride;  // elements per layer = n_pages*page_size*n_kv_heads*head_dim
};

__device__ __forceinline__ int64_t kv_token_offset(const KvView& kv, int seq, int pos) {
  int page = kv.page_table[(int64_t)seq * kv.max_pages + pos / kv.page_size];
  return ((int64_t)page * kv.page_size + pos % kv.page_size) * kv.n_kv_heads * kv.head_dim;
}
__device__ __forceinline__ int kv_capacity(const KvView& kv) { return kv.page_size * kv.max_pages; }

// Row descriptors of one pass (R rows per sequence, B sequences), device arrays in the workspace
struct RowDesc {
  int32_t* tok;    // [B*R] token id of the row
  int32_t* pos;    // [B*R] rotary position
  int32_t* slot;   // [B*R] logical KV position the row's K/V are written to, -1 = inactive row
  uint64_t* mask;  // [B*R] visible speculative slots: bit j <=> logical position len+j
  int32_t* nspec;  // [B]   speculative slots in use after this pass (keys len .. len+nspec-1 exist)
};

// ---- launchers (kernels_*.hip) ----------------------------------------------------------------
// h = E[tok]; bf16 models also get the first RMSNorm's input: h*g0 as two bf16 terms (layout: act_offset with ncg) and ssq[rows] = sum h^2;
// and the rotary table of the rows' positions, table[rows][head_dim/2] = (cos, sin)
hipError_t launch_embed(int dtype, const void* E, const int32_t* tok, float* h, int rows, int d, int vocab, const float* g0,
                        void* planes, float* ssq, const int32_t* pos, float2* table, int head_dim, float theta, int ncg, hipStream_t s);
// out = rmsnorm(h) * g, written as hi/lo bf16 planes [2][rows][d] (dtype 1) or f32 [rows][d] (dtype 0)
hipError_t launch_rmsnorm(int dtype, const float* h, const float* g, void* out, int rows, int d, float eps, hipStream_t s);
// q: [rows][q_stride] float32 with head h at column h*head_dim; counters: zeroed ints [B][n_heads][ceil(R/8)], used by
// the last workgroup of an item, which merges the key splits (bf16 models: in passes of few rows, else a kernel of its own does)
hipError_t launch_attention(int dtype, const float* q, int q_stride, const RowDesc& rd, KvView kv, int layer, int B, int R, int n_heads,
                            float* partial, int n_splits, int* counters, void* out, int ncg, hipStream_t s);
// bf16 models (kernels_attn_mfma.hip): half-precision cache, output = bf16 hi / lo terms (layout: act_offset with ncg);
// n_splits = upper bound on the key splits (the kernel uses fewer for short contexts); counters (zeroed, [B][n_kv_heads], or null): a pass
// of few rows merges its key splits in the same launch
hipError_t launch_attention_mfma(const float* q, int q_stride, const RowDesc& rd, KvView kv, int layer, int B, int R, int n_heads,
                                 float* partial, int n_splits, void* out, int ncg, hipStream_t s, int* counters = nullptr);
// the same for a chunk of a prompt: any number of rows per sequence, row r sees the committed context and rows 0 .. r
hipError_t launch_attention_prompt(const float* q, int q_stride, const RowDesc& rd, KvView kv, int layer, int B, int R, int n_heads, float* partial,
                                   int n_splits, void* out, int ncg, hipStream_t s);
// lse[row] from per-strip (max, sum exp) partials [rows][NP]
hipError_t launch_lse_finish(const float* lse_part, float* lse, int rows, int NP, hipStream_t s);
// lse as above for B*M rows, plus logp_cond[s][c] = logits[s][parent(c)][tok(c)] - lse[s][parent(c)] (0 for c = 0)
hipError_t launch_lse_gather(const float* lse_part, float* lse, int B, int M, int NP, const float* logits, int V, const int32_t* parent,
                             const int32_t* tok, float* logp_cond, hipStream_t s);
hipError_t launch_copy(const void* src, void* dst, int64_t bytes, hipStream_t s);
hipError_t launch_row_lse(const float* logits, float* lse, int rows, int vocab, hipStream_t s);

// most key splits of a float32 model's attention in a context of that many keys
int f32_attention_splits(int B, int n_heads, int R, int max_context);
size_t attention_partial_floats(int B, int R, int n_heads, int head_dim, int n_splits);

}  // namespace mtad
