// Tree-masked paged attention of float32 models (Section 3.3: tree attention gives every tree token its conditional likelihood in one
// pass), and the launcher that picks the kernel of a pass.  Every row sees the whole committed cache of its sequence plus the
// speculative rows named in its ancestor mask.  Everything is float32 arithmetic.
//
// Grid = (key split, query head x chunk of 8 rows, sequence), eight waves a workgroup.  A wave works on blocks of 64 keys for four of
// the rows, with K and V of a block in registers, all its requests on their way together, and nothing staged in LDS:
//   scores   lane (g, c) holds dims 4c .. 4c + 3 (and 64 further on) of keys 4j + g, j = 0 .. 15: sixteen partial dot products, which a
//            reduction over the 16 lanes of a row that halves the keys a lane is left with at each step turns into the score of
//            key 4c + g in lane (g, c);
//   output   the same layout of V; p of key 4j + g is the value of lane j of the row, a data-parallel move.
// Waves 2b and 2b + 1 take key block b of every four and half of the rows each; the four blocks' waves meet in LDS.  Contexts of more
// than 256 keys are cut into splits; the workgroup that arrives last for a (sequence, head, chunk) merges them in split order.
// Bound by latency: a launch, the length, the page, the block and its arithmetic are a chain.  us, tiles staged in LDS and a thread per
// (key, rows) before / here: 5 rows x 4 heads x 64, 82 keys 9.2 / 6.3 (in a pass 11.1 / 6.5); one row x 8 heads, 300 keys 12.1 / 6.7; 5 rows x
// 4 heads x 128, 4096 keys 52.7 / 20.7; 3 x 57 rows x 8 heads x 64, 900 keys (arithmetic) 38.5 / 38.6.
// A compute unit holds one workgroup (212 registers, eight waves), and a wave's next block costs less than a workgroup's start and a share of the
// merge: no more splits than give every compute unit one.  us of a pass of four narrow layers, splits for four workgroups a compute unit / two / one / half
// of them: 16 x 9 rows x 8 heads x 64, 700 keys 290 / 255 / 212 / 212; 16 x 5 rows, 1500 keys 256 / 248 / 215 / 265; 4 x 25 rows, 1500 keys 242 / 228 / 207 / 244; one
// sequence of 57 rows, 1500 keys 172 / 171 / 147 / 170; 5 rows, 700 keys (32 workgroups a split) alike.  (At one a compute unit, chunks and query
// heads that share keys are KV heads apart in the grid, so that they mostly are on one XCD and its cache has the keys once: 2 x 57 rows x 8 heads x 128,
// 8100 keys 817 / 595, 8 x 9 rows, 4100 keys 562 / 488, 700 keys 224 / 208.)
#include "attn_mfma_device.h"
#include "common.h"

namespace mtad {

namespace {

constexpr int F32_ROWS = 8, F32_BLOCK = 64, F32_BLOCKS = 4;  // rows of a workgroup, keys of a block, blocks side by side
constexpr int F32_THREADS = 2 * F32_BLOCKS * 64, HALF_ROWS = F32_ROWS / 2;

__device__ __forceinline__ int f32_splits(int ktot, int n_splits) {
  return max(1, min(n_splits, (ktot + F32_BLOCKS * F32_BLOCK - 1) / (F32_BLOCKS * F32_BLOCK)));
}
template <int J>
__device__ __forceinline__ int row_lane(int v) {  // the value of lane J of the row of 16
  return __builtin_amdgcn_update_dpp(0, v, 0x150 + J, 0xf, 0xf, true);
}
// One step of scatter_sum: of 2N partial sums a lane keeps the N whose number has the lane's bit N and adds the partner's, N lanes away
// (distance 8: a rotation; 4: a mirror of eight lanes and one of four; 2 and 1: a permutation of four lanes).
template <int N>
__device__ __forceinline__ void halve(float* y, int c) {
#pragma unroll
  for (int j = 0; j < N; ++j) {
    const float keep = (c & N) ? y[j + N] : y[j];
    const int give = __float_as_int((c & N) ? y[j] : y[j + N]);
    int got;
    if constexpr (N == 8) got = __builtin_amdgcn_update_dpp(0, give, 0x128, 0xf, 0xf, true);
    if constexpr (N == 4) got = __builtin_amdgcn_update_dpp(0, __builtin_amdgcn_update_dpp(0, give, 0x141, 0xf, 0xf, true), 0x1B, 0xf, 0xf, true);
    if constexpr (N == 2) got = __builtin_amdgcn_update_dpp(0, give, 0x4E, 0xf, 0xf, true);
    if constexpr (N == 1) got = __builtin_amdgcn_update_dpp(0, give, 0xB1, 0xf, 0xf, true);
    y[j] = keep + __int_as_float(got);
  }
}
// x[j] summed over the 16 lanes of a row, for j = the lane's number in its row (c)
__device__ __forceinline__ float scatter_sum(float (&x)[16], int c) {
  halve<8>(x, c);
  halve<4>(x, c);
  halve<2>(x, c);
  halve<1>(x, c);
  return x[0];
}
template <typename F, int... J>
__device__ __forceinline__ void each_of(F f, std::integer_sequence<int, J...>) {
  (f(std::integral_constant<int, J>{}), ...);
}
template <typename F>
__device__ __forceinline__ void each16(F f) {
  each_of(f, std::make_integer_sequence<int, 16>{});
}

template <int HD>
__global__ __launch_bounds__(F32_THREADS) __attribute__((amdgpu_waves_per_eu(2))) void tree_attn_f32_kernel(
    const float* __restrict__ q, int q_stride, RowDesc rd, KvView kv, int layer, int R, int n_heads, int group, int n_chunks, float scale,
    float* __restrict__ partial, int n_splits, int* __restrict__ counters, float* __restrict__ out) {
  constexpr int E = HD / 64;  // float4s per lane of a key or a query
  __shared__ __attribute__((aligned(16))) float o_s[F32_BLOCKS][F32_ROWS][HD];
  __shared__ float m_s[F32_BLOCKS][F32_ROWS], l_s[F32_BLOCKS][F32_ROWS];
  __shared__ int last_s;
  const int t = threadIdx.x, lane = t & 63, c = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6), kb = wave >> 1;
  const int KVH = kv.n_kv_heads, kv_head = blockIdx.y % KVH, rest = blockIdx.y / KVH;
  const int split = blockIdx.x, head = kv_head * group + rest % group, chunk = rest / group, seq = blockIdx.z;
  const int nrows = min(F32_ROWS, R - chunk * F32_ROWS), half = (nrows + 1) >> 1;
  const int r0 = (wave & 1) * half, nr = (wave & 1) ? nrows - half : half;  // this wave's rows of the chunk
  const int row0 = seq * R + chunk * F32_ROWS + r0;
  const int cap = kv_capacity(kv);

  // what does not depend on the length first: the place of this lane's key of the first block, the queries
  // (all kernel arguments at once; left to itself the compiler fetches them in rounds, each a trip to memory)
  asm volatile("" ::"s"(q), "s"(q_stride), "s"(rd.nspec), "s"(rd.mask), "s"(kv.k), "s"(kv.v), "s"(kv.page_table), "s"(kv.len), "s"(kv.page_size), "s"(kv.max_pages),
               "s"(kv.n_pages), "s"(kv.n_kv_heads), "s"(kv.layer_stride), "s"(layer), "s"(R), "s"(n_heads), "s"(n_splits), "s"(n_chunks), "s"(group), "s"(out));
  auto key_of = [&](int block) { return min(block * F32_BLOCK + 4 * c + g, cap - 1); };
  const int block0 = split * F32_BLOCKS + kb;
  const int page0 = kv.page_table[(int64_t)seq * kv.max_pages + key_of(block0) / kv.page_size];
  float4 qv[HALF_ROWS][E];
  unsigned long long mask[HALF_ROWS];
#pragma unroll
  for (int r = 0; r < HALF_ROWS; ++r) {
    const int row = min(row0 + r, seq * R + R - 1);
    mask[r] = rd.mask[row];
#pragma unroll
    for (int e = 0; e < E; ++e) qv[r][e] = *(const float4*)(q + (int64_t)row * q_stride + head * HD + e * 64 + 4 * c);
  }
  int tok = ((page0 < 0 || page0 >= kv.n_pages) ? 0 : page0) * kv.page_size + key_of(block0) % kv.page_size;
  const int len = kv.len[seq], ktot = attn_keys(kv, rd, seq), eff = f32_splits(ktot, n_splits);
  if (split >= eff) return;
  const int blocks = nr > 0 ? (ktot + F32_BLOCK - 1) / F32_BLOCK : 0;

  const int64_t tok_stride = (int64_t)kv.n_kv_heads * HD;
  const int64_t at = (int64_t)layer * kv.layer_stride + (int64_t)kv_head * HD + 4 * c;
  const float *const kbase = (const float*)kv.k + at, *const vbase = (const float*)kv.v + at;
  float m_run[HALF_ROWS], l_run[HALF_ROWS];
  float4 acc[HALF_ROWS][E];
#pragma unroll
  for (int r = 0; r < HALF_ROWS; ++r) {
    m_run[r] = -INFINITY;
    l_run[r] = 0.f;
#pragma unroll
    for (int e = 0; e < E; ++e) acc[r][e] = make_float4(0.f, 0.f, 0.f, 0.f);
  }
#pragma unroll 1
  for (int b = block0; b < blocks; b += eff * F32_BLOCKS) {
    float4 kf[16][E], vf[16][E];
    const int tok_b = tok;
    auto request = [&](float4 (&f)[16][E], const float* base) {
      each16([&](auto J) {
        constexpr int j = J;
        const float* const p = base + (int64_t)row_lane<j>(tok_b) * tok_stride;
#pragma unroll
        for (int e = 0; e < E; ++e) f[j][e] = *(const float4*)(p + e * 64);
      });
    };
    request(kf, kbase);
    if constexpr (E == 1) request(vf, vbase);  // (two float4s per key and lane: no room for V beside K)
    const int next = b + eff * F32_BLOCKS;
    if (next < blocks) tok = token_index(kv, seq, key_of(next));
    const int key = b * F32_BLOCK + 4 * c + g;
    float p[HALF_ROWS];
#pragma unroll
    for (int r = 0; r < HALF_ROWS; ++r) {
      p[r] = 0.f;
      if (r < nr) {  // uniform over the wave
        float x[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) {
          x[j] = qv[r][0].x * kf[j][0].x;
          x[j] = fmaf(qv[r][0].y, kf[j][0].y, x[j]);
          x[j] = fmaf(qv[r][0].z, kf[j][0].z, x[j]);
          x[j] = fmaf(qv[r][0].w, kf[j][0].w, x[j]);
          if constexpr (E == 2) {
            x[j] = fmaf(qv[r][1].x, kf[j][1].x, x[j]);
            x[j] = fmaf(qv[r][1].y, kf[j][1].y, x[j]);
            x[j] = fmaf(qv[r][1].z, kf[j][1].z, x[j]);
            x[j] = fmaf(qv[r][1].w, kf[j][1].w, x[j]);
          }
        }
        float s = scatter_sum(x, c) * scale;
        const bool sees = key < len || (key < ktot && ((mask[r] >> (key - len)) & 1ull));
        s = sees ? s : -INFINITY;
        const float m_new = fmaxf(m_run[r], wave_max(s)), m_sub = m_new == -INFINITY ? 0.f : m_new;
        const float alpha = expf(m_run[r] - m_sub);
        p[r] = expf(s - m_sub);
        l_run[r] = l_run[r] * alpha + p[r];
        m_run[r] = m_new;
#pragma unroll
        for (int e = 0; e < E; ++e) {
          acc[r][e].x *= alpha; acc[r][e].y *= alpha; acc[r][e].z *= alpha; acc[r][e].w *= alpha;
        }
      }
    }
    if constexpr (E == 2) request(vf, vbase);
    if (b * F32_BLOCK + F32_BLOCK > ktot) {  // uniform: what lies past the last key is not read into any sum
#pragma unroll
      for (int j = 0; j < 16; ++j)
        if (b * F32_BLOCK + 4 * j + g >= ktot) {
#pragma unroll
          for (int e = 0; e < E; ++e) vf[j][e] = make_float4(0.f, 0.f, 0.f, 0.f);
        }
    }
#pragma unroll
    for (int r = 0; r < HALF_ROWS; ++r)
      if (r < nr) {
        each16([&](auto J) {
          constexpr int j = J;
          const float pj = __int_as_float(row_lane<j>(__float_as_int(p[r])));
#pragma unroll
          for (int e = 0; e < E; ++e) {
            acc[r][e].x = fmaf(pj, vf[j][e].x, acc[r][e].x);
            acc[r][e].y = fmaf(pj, vf[j][e].y, acc[r][e].y);
            acc[r][e].z = fmaf(pj, vf[j][e].z, acc[r][e].z);
            acc[r][e].w = fmaf(pj, vf[j][e].w, acc[r][e].w);
          }
        });
      }
  }
#pragma unroll
  for (int r = 0; r < HALF_ROWS; ++r)
    if (r < nr) {
      const float l = wave_sum(l_run[r]);
      if (lane == 0) {
        m_s[kb][r0 + r] = m_run[r];
        l_s[kb][r0 + r] = l;
      }
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const float4 a = acc[r][e];
        const float4 o = make_float4(xsum<32>(xsum<16>(a.x)), xsum<32>(xsum<16>(a.y)), xsum<32>(xsum<16>(a.z)), xsum<32>(xsum<16>(a.w)));
        if (g == 0) *(float4*)&o_s[kb][r0 + r][e * 64 + 4 * c] = o;
      }
    }
  __syncthreads();
  // the blocks' waves, added in order: thread (row, dim)
  const int64_t prow = ((int64_t)seq * n_heads + head) * R + chunk * F32_ROWS;  // of row 0 among the partial results
  float* const orow = out + (int64_t)(seq * R + chunk * F32_ROWS) * n_heads * HD + (int64_t)head * HD;
#pragma unroll
  for (int i = t; i < F32_ROWS * HD; i += F32_THREADS) {
    const int r = i / HD, d = i % HD;
    if (r >= nrows) break;
    float M = m_s[0][r], L = 0.f, o = 0.f;
#pragma unroll
    for (int w = 1; w < F32_BLOCKS; ++w) M = fmaxf(M, m_s[w][r]);
#pragma unroll
    for (int w = 0; w < F32_BLOCKS; ++w) {
      const float e = m_s[w][r] == -INFINITY ? 0.f : expf(m_s[w][r] - M);
      L += l_s[w][r] * e;
      o += o_s[w][r][d] * e;
    }
    if (eff == 1) {
      orow[(int64_t)r * n_heads * HD + d] = L > 0.f ? o / L : 0.f;
    } else {  // (max, sum, output) of the split, for the workgroup that arrives last: write-through stores, as the XCDs' caches are not coherent
      float* const p = partial + ((prow + r) * n_splits + split) * (HD + 2);
      st4<true>(p + 2 + d, o);
      if (d == 0) {
        st4<true>(p, M);
        st4<true>(p + 1, L);
      }
    }
  }
  if (eff == 1) return;
  __builtin_amdgcn_s_waitcnt(0);  // the stores have been acknowledged
  __syncthreads();
  if (t == 0) {
    int* const cn = counters + ((int64_t)seq * n_heads + head) * n_chunks + chunk;
    const int prev = __hip_atomic_fetch_add(cn, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    last_s = prev == eff - 1;
    if (prev == eff - 1) __hip_atomic_store(cn, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);  // clean for the next launch
  }
  __syncthreads();
  if (!last_s) return;
#pragma unroll
  for (int i = t; i < F32_ROWS * HD; i += F32_THREADS) {
    const int r = i / HD, d = i % HD;
    if (r >= nrows) break;
    const float* const p = partial + (prow + r) * n_splits * (HD + 2);
    float M = -INFINITY, L = 0.f, o = 0.f;
    for (int s0 = 0; s0 < eff; s0 += 8) {  // in split order, eight splits' loads in flight at a time
      float mm[8], ll[8], oo[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const float* const ps = p + (int64_t)min(s0 + j, eff - 1) * (HD + 2);
        mm[j] = ld4<true>(ps);
        ll[j] = ld4<true>(ps + 1);
        oo[j] = ld4<true>(ps + 2 + d);
      }
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        if (s0 + j >= eff || mm[j] == -INFINITY) continue;
        const float Mn = fmaxf(M, mm[j]);
        const float ws = M == -INFINITY ? 0.f : expf(M - Mn), wj = expf(mm[j] - Mn);
        L = L * ws + ll[j] * wj;
        o = o * ws + oo[j] * wj;
        M = Mn;
      }
    }
    orow[(int64_t)r * n_heads * HD + d] = L > 0.f ? o / L : 0.f;
  }
}

template <int HD>
hipError_t run_f32(const float* q, int q_stride, const RowDesc& rd, const KvView& kv, int layer, int B, int R, int n_heads, float* partial, int n_splits,
                   int* counters, void* out, hipStream_t s) {
  const int n_chunks = (R + F32_ROWS - 1) / F32_ROWS;
  hipLaunchKernelGGL((tree_attn_f32_kernel<HD>), dim3(n_splits, n_heads * n_chunks, B), dim3(F32_THREADS), 0, s, q, q_stride, rd, kv, layer, R, n_heads, n_heads / kv.n_kv_heads,
                     n_chunks, 1.0f / sqrtf((float)HD), partial, n_splits, counters, (float*)out);
  return hipGetLastError();
}

}  // namespace

int f32_attention_splits(int B, int n_heads, int R, int max_context) {
  const int items = B * n_heads * ((R + F32_ROWS - 1) / F32_ROWS), fill = (256 + items - 1) / items, most = (max_context + F32_BLOCKS * F32_BLOCK - 1) / (F32_BLOCKS * F32_BLOCK);
  const int s = fill < most ? fill : most;
  return s < 1 ? 1 : s > 32 ? 32 : s;  // (32: what the exchange buffer is made for)
}

size_t attention_partial_floats(int B, int R, int n_heads, int head_dim, int n_splits) {
  return (size_t)B * R * n_heads * n_splits * (head_dim + 2);
}

hipError_t launch_attention(int dtype, const float* q, int q_stride, const RowDesc& rd, KvView kv, int layer, int B, int R, int n_heads,
                            float* partial, int n_splits, int* counters, void* out, int ncg, hipStream_t s) {
  if (B * R <= 0) return hipSuccess;
  const int hd = kv.head_dim;
  if (dtype == 1) return launch_attention_mfma(q, q_stride, rd, kv, layer, B, R, n_heads, partial, n_splits, out, ncg, s, counters);
  if (dtype == 0 && hd == 128) return run_f32<128>(q, q_stride, rd, kv, layer, B, R, n_heads, partial, n_splits, counters, out, s);
  if (dtype == 0 && hd == 64) return run_f32<64>(q, q_stride, rd, kv, layer, B, R, n_heads, partial, n_splits, counters, out, s);
  return hipErrorInvalidValue;
}

}  // namespace mtad

// Host side only, for the tests.
extern "C" int mtad_test_f32_attention_splits(int batch, int n_heads, int rows, int max_context) {
  return mtad::f32_attention_splits(batch, n_heads, rows, max_context);
}
