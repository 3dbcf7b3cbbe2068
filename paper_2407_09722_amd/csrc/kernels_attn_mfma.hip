// Tree-masked paged attention for bf16 models (half-precision K/V cache), few query rows per sequence
// (Section 3.3: tree attention gives every tree token its conditional likelihood in one pass): the stand-alone kernels.
// The work item itself (tile loop on the matrix cores, online softmax, merge of the waves) is in attn_mfma_device.h.
//
// Work item = (key split, KV head, chunk of 16 or 32 (query head, row) pairs, sequence) = one workgroup of AW waves (4 in
// all configurations used; 8 measured no faster).  A context of fewer than 2 x waves x 32 keys is one workgroup,
// which writes the attention output itself: no exchange through global memory.  Longer contexts are cut into splits
// (at least one tile per wave each, at most as many as fill the machine once, or every resident slot where once is an
// uneven fill); every split leaves (max, sum, output)
// per row in global memory (same partial layout as the generic kernel) and a small second kernel, one wave per row,
// merges them in split order.  More than 32 pairs on a KV head, and prompts of any number of rows, go to a kernel whose waves share
// the tiles (tree_attn_rows_kernel).
#include "attn_mfma_device.h"
#include "common.h"

#include <type_traits>

namespace mtad {

namespace {

constexpr int FEW_ROWS = 64;  // (sequence, query head, row) triples of a pass that merges its key splits in the attention launch

int device_cus() {
  static const int n_cus = [] {
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) cus = 0;
    return cus > 0 ? cus : 256;
  }();
  return n_cus;
}

// A workgroup's place among key splits, KV heads, sequences (and chunks of rows, the slowest).  Workgroups go to the XCDs in turn, and a sequence
// may use only the first few of the splits a launch offers.  Where the launch offers no more than one workgroup a compute unit, the splits
// of an item are neighbours.  Where it offers more (spread), those in use would crowd on some XCDs (offered 8, in use 4: on half of them), so
// the splits run slowest, and the KV heads are turned by sequence and split: a head's rows lie at a fixed place in every token of the cache, and
// an XCD that reads all heads in turn is the faster one.  (With one workgroup a compute unit and one split that writes its output itself,
// turned heads were slower, 32 x 5 rows x 64 heads on 8 x 128, 60 keys 217 / 224.  With few items their chunks, which
// share keys, would go to different XCDs: 33 rows x 16 heads on 2 x 64, 4100 keys 168 / 176.)
// us of a pass of four narrow layers, splits fastest / slowest / slowest and heads turned: 8 x one row x 12 heads x 64, 2064 keys 163 / 141 / 141;
// 4 x one row x 40 heads x 64, 1100 keys 163 / 146 / 144, 2064 keys 211 / 197 / 186; 4 x 33 rows x 40 heads x 128, 300 keys 275 / 263 / 262; 8 x one
// row x 40 heads x 128, 2064 keys 432 / - / 410.
struct AttnPlace {
  int split, g, seq, chunk;
};
__host__ __device__ constexpr AttnPlace attn_place(bool spread, int KVH, int x, int y, int z) {  // grid: attn_grid()
  const int split = spread ? z : x, head = spread ? x : y, seq = spread ? y : z;
  return {split, spread ? (head + seq + split) % KVH : head, seq, 0};
}
bool spread_splits(int offered, int items) { return 4 * items > device_cus() && offered * items > device_cus(); }
dim3 attn_grid(bool spread, int gx, int KVH, int B) { return spread ? dim3(KVH, B, gx) : dim3(gx, KVH, B); }
__host__ __device__ constexpr AttnPlace rows_place(int splits, int KVH, int B, int x, int y) {  // splits: 0 if spread; grid: rows_grid()
  const int split = splits ? x % splits : y, item = splits ? x / splits : x, seq = item / KVH % B;
  return {split, (splits ? item : item + seq + split) % KVH, seq, item / (KVH * B)};
}
dim3 rows_grid(bool spread, int gx, int items) { return spread ? dim3(items, gx) : dim3(items * gx); }

template <int HD, int NRG, int AW>
__global__ __launch_bounds__(AW * 64) __attribute__((amdgpu_waves_per_eu(2))) void tree_attn_mfma_kernel(const float* __restrict__ q, int q_stride, RowDesc rd, KvView kv, int layer,
                                                               int B, int R, int n_heads, float scale, float* __restrict__ partial,
                                                               int n_splits, bf16_t* __restrict__ out, int want_splits, int ncg, bool spread) {
  using Smem = MfmaAttnSmem<HD, NRG, AW>;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  Smem& sm = *reinterpret_cast<Smem*>(smem_raw);
  // the kernels with registers to spare (head dim 64, or a single row group) hold two register sets for K and V
  constexpr int NSET = (HD == 64 || NRG == 1) ? 2 : 1;
  const AttnPlace at = attn_place(spread, kv.n_kv_heads, blockIdx.x, blockIdx.y, blockIdx.z);
  tree_attn_item<HD, NRG, AW, NSET, AW * 64, false>(sm, q, q_stride, rd, kv, layer, B, R, n_heads, 1, scale, partial, n_splits, out, want_splits, ncg, at.split,
                                                    at.g, 0, at.seq, (int)threadIdx.x);
}

// The same item for passes of few rows in all (small models): the key split that arrives last for an item merges its rows,
// one wave a row, instead of a launch of its own for a handful of waves.  Bound by latency: 12 heads x 64, one row, 256 keys:
// 9.0 us against 6.3 + 3.1 in two launches and the gap between them (12 layers: 323 -> 311 us).
// counters: one zeroed word per item, left zeroed.  At most ATTN_WAVES rows an item.
template <int HD>
__global__ __launch_bounds__(ATTN_WAVES * 64) __attribute__((amdgpu_waves_per_eu(2))) void tree_attn_few_kernel(
    const float* __restrict__ q, int q_stride, RowDesc rd, KvView kv, int layer, int B, int R, int n_heads, float scale, float* __restrict__ partial, int n_splits,
    bf16_t* __restrict__ out, int want_splits, int ncg, bool spread, int* __restrict__ counters) {
  __shared__ MfmaAttnSmem<HD, 1, ATTN_WAVES> sm;
  __shared__ int last_s;
  const AttnPlace at = attn_place(spread, kv.n_kv_heads, blockIdx.x, blockIdx.y, blockIdx.z);
  const int split = at.split, g = at.g, seq = at.seq, t = threadIdx.x;
  const int eff = tree_attn_item<HD, 1, ATTN_WAVES, 2, ATTN_WAVES * 64, true>(sm, q, q_stride, rd, kv, layer, B, R, n_heads, 1, scale, partial, n_splits, out,
                                                                            want_splits, ncg, split, g, 0, seq, t);
  if (eff == 1 || split >= eff) return;  // uniform: the item wrote its output itself, or there was no such split
  __builtin_amdgcn_s_waitcnt(0);  // the partial results have been acknowledged
  __syncthreads();
  if (t == 0) {
    int* const c = counters + seq * kv.n_kv_heads + g;
    const int prev = __hip_atomic_fetch_add(c, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    last_s = prev == eff - 1;
    if (prev == eff - 1) __hip_atomic_store(c, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);  // clean for the next launch
  }
  __syncthreads();
  if (!last_s) return;
  const int G = n_heads / kv.n_kv_heads;
  const int p = t >> 6;
  if (p < G * R) {
    const int head = g * G + p / R, row = p % R;
    attn_merge_row<HD, true>(partial + (((int64_t)seq * n_heads + head) * R + row) * n_splits * (HD + 2), eff, out, ncg, B * R, n_heads * HD, seq * R + row, head,
                             t & 63);
  }
}

// ---- items of many rows ---------------------------------------------------------------------------------------------
// Work item = (key split, KV head, chunk of 16 RW (query head, row) pairs, sequence) = one workgroup of RW = 3 or 4 waves.  A wave owns
// a row group of 16, its query fragments (hi and lo halves) in registers, and works on every tile of the item; K and V
// tiles lie in two slots in LDS that all waves read, so that they come from memory once for 16 RW rows, and nothing has to be
// merged between waves.  Tiles go from memory to LDS without passing registers (16 bytes per lane, four or eight cache rows an
// instruction), the next one while this one is worked on; one barrier a tile: it ends the reads of the slot that is refilled and
// says that every wave's share of the tile has arrived.
// Where the 16-byte chunks of a row lie is turned by its key, so that 16 keys' chunk c (an operand of K) and the 32-byte pieces of
// eight keys (a transposing read of V) fall into different banks.
// What bounds it: a tile costs a wave as many clocks of LDS reads (K and V once per 16 rows) as of matrix instructions, and the
// waves of a compute unit overlap the two only in part.  us with the merge of the splits, in items of 32 or 48 rows whose four
// waves have tiles of their own (above) / here: prompts of 2047 rows x 32 heads x 128 146 / 90, 4 x 509 x 40 heads 96 / 48, 4 x 512 rows x
// 32 heads on 4 x 64 48 / 25; trees: 4 x 41 rows x 40 heads x 128, 4100 keys 91 / 86 (3.9 TB/s; requests alone 63, arithmetic on
// cached tiles alone 60), 8 heads on a key head 81 / 56; 4 x 8 rows x 32 heads on 4 x 64, 4100 keys 20.4 / 16.1; 40 rows x 32 heads x 64, 900
// keys 16.0 / 11.3.  Up to 32 pairs a KV head (there / here with two waves): 17 rows x 32 heads x 128, 2064 keys 19.7 / 19.6; 8 x 30 rows x 16
// heads, 700 keys 23.0 / 24.5; 4 x 20 rows x 32 heads x 64, 4000 keys 43.7 / 47.9: they stay above.
// Measured and not better: two row groups a wave (prompt of 2047 rows 101, half the LDS reads but twice the work of the longest item);
// three or four slots; tiles of 64 keys for head dim 128 (93) or of 32 for 64 (26 instead of 25).
constexpr int ROWS_WAIT_ALL = 0x0070;  // s_waitcnt: no vector memory operation and no LDS operation outstanding
constexpr int LOOK_KEYS = 512;  // keys whose places in the cache are looked up together

template <int HD, int RW>
struct RowsShape {
  static constexpr int RTK = HD == 128 ? 32 : 64;     // keys per tile (8 KiB of K and of V)
  static constexpr int TOK_TILES = LOOK_KEYS / RTK;  // tiles looked up together
  static constexpr int CPR = HD / 8;          // 16-byte chunks of a cache row
  static constexpr int KPI = 64 / CPR;        // keys one request covers
  static constexpr int GROUPS = RTK / KPI;    // requests for K (and as many for V) per tile
  static constexpr int TILE = RTK * HD * 2, SLOT = 2 * TILE;
  static constexpr int LDS = 2 * SLOT + 2 * TOK_TILES * RTK * 4;
  static constexpr int WAVES = HD == 128 ? 3 : 4;  // per SIMD
  static constexpr int LOOK = (TOK_TILES * RTK + RW * 64 - 1) / (RW * 64);  // keys a thread looks up per block of tiles
};

template <int HD, int RW, bool CAUSAL>
__global__ __launch_bounds__(RW * 64) __attribute__((amdgpu_waves_per_eu(RowsShape<HD, RW>::WAVES))) void tree_attn_rows_kernel(
    const float* __restrict__ q, int q_stride, RowDesc rd, KvView kv, int layer, int B, int R, int n_heads, int n_chunks, float scale,
    float* __restrict__ partial, int n_splits, bf16_t* __restrict__ out, int want_splits, int ncg, int splits) {
  using Sh = RowsShape<HD, RW>;
  constexpr int KS = HD / 32, DB = HD / 16, CPR = Sh::CPR, KPI = Sh::KPI, GROUPS = Sh::GROUPS, TILE = Sh::TILE, SLOT = Sh::SLOT, LOOK = Sh::LOOK, RTK = Sh::RTK, TOK_TILES = Sh::TOK_TILES, NB = RTK / 16;
  extern __shared__ __attribute__((aligned(256))) unsigned char ring[];
  int* const tokens = (int*)(ring + 2 * SLOT);  // [2][TOK_TILES][RTK]

  const int t = threadIdx.x, lane = t & 63, srow = lane & 15, sg4 = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  // (all kernel arguments at once; left to itself the compiler fetches them in rounds, each a trip to memory)
  asm volatile("" ::"s"(q), "s"(q_stride), "s"(rd.nspec), "s"(rd.mask), "s"(kv.k), "s"(kv.v), "s"(kv.page_table), "s"(kv.len), "s"(kv.page_size), "s"(kv.max_pages),
               "s"(kv.n_pages), "s"(kv.n_kv_heads), "s"(kv.layer_stride), "s"(layer), "s"(R), "s"(n_heads), "s"(n_splits), "s"(n_chunks), "s"(splits));
  const int KVH = kv.n_kv_heads, G = n_heads / KVH;
  const AttnPlace at = rows_place(splits, KVH, B, blockIdx.x, blockIdx.y);
  const int split = at.split, g = at.g, seq = at.seq, chunk = CAUSAL ? n_chunks - 1 - at.chunk : at.chunk;  // a prompt's items that see the most keys first
  const int pairs = G * R, pair0 = chunk * (RW * 16), pair_end = min(pairs, pair0 + RW * 16);  // pair p = query head p / R of the group, row p % R
  const int wp0 = pair0 + wave * 16, wp_end = min(pair_end, wp0 + 16);                      // this wave's
  const bool rowless = wp0 >= pair_end;

  const int len = kv.len[seq], ktot = attn_keys(kv, rd, seq, CAUSAL), eff = attn_splits(ktot, n_splits, want_splits);
  if (split >= eff) return;
  // keys the item sees, keys the wave sees, keys all the wave's rows see
  auto last_row = [&](int p0, int p1) { return p0 / R == (p1 - 1) / R ? (p1 - 1) % R : R - 1; };
  int kend = ktot, wend = ktot, all = len;
  if constexpr (CAUSAL) {
    kend = min(ktot, len + 1 + last_row(pair0, pair_end));
    if (!rowless) {
      wend = min(ktot, len + 1 + last_row(wp0, wp_end));
      all = len + 1 + (wp0 / R == (wp_end - 1) / R ? wp0 % R : 0);
    }
  }
  all = min(all, wend);
  const int tiles = (kend + RTK - 1) / RTK, n_my = tiles > split ? (tiles - split + eff - 1) / eff : 0;  // tiles split, split + eff, ..

  // keys of tiles block * TOK_TILES .. of this split, LOOK per thread; past the end the last key
  auto key_of = [&](int block, int e) { return max(0, min((split + (block * TOK_TILES + e / RTK) * eff) * RTK + e % RTK, kend - 1)); };
  int page[LOOK];
  auto look_up = [&](int block) {
#pragma unroll
    for (int j = 0; j < LOOK; ++j) page[j] = kv.page_table[(int64_t)seq * kv.max_pages + key_of(block, t + j * (RW * 64)) / kv.page_size];
  };
  auto put = [&](int block) {
#pragma unroll
    for (int j = 0; j < LOOK; ++j) {
      const int e = t + j * (RW * 64), pg = (page[j] < 0 || page[j] >= kv.n_pages) ? 0 : page[j];
      if (e < TOK_TILES * RTK) tokens[(block & 1) * (TOK_TILES * RTK) + e] = pg * kv.page_size + key_of(block, e) % kv.page_size;
    }
  };
  look_up(0);

  // the wave's queries: lane (sg4, srow) of fragment ks holds dims ks * 32 + sg4 * 8 .. + 7 of row srow; rows that do not exist are zeros
  half8 qh[1][KS], ql[1][KS];
  unsigned long long rmask[1];  // CAUSAL: the first key the row does not see
  {
    const int p = wp0 + srow;
    const bool live = p < wp_end;
    const int pc = live ? p : 0, row = pc % R;
    const float* const qp = q + (int64_t)(seq * R + row) * q_stride + (int64_t)(g * G + pc / R) * HD + sg4 * 8;
    if constexpr (CAUSAL) rmask[0] = live ? (unsigned)(len + 1 + row) : 0u;
    else rmask[0] = live ? rd.mask[seq * R + row] : 0ull;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      typedef float floatx8_t __attribute__((ext_vector_type(8)));
      const float4 a = *(const float4*)(qp + ks * 32), b = *(const float4*)(qp + ks * 32 + 4);
      const floatx8_t x = live ? floatx8_t{a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w} : floatx8_t{};
      qh[0][ks] = __builtin_convertvector(x, half8);
      ql[0][ks] = __builtin_convertvector(x - __builtin_convertvector(qh[0][ks], floatx8_t), half8);
    }
  }
  put(0);
  __syncthreads();

  typedef const __attribute__((address_space(1))) uint32_t* GlobalWords;
  typedef __attribute__((address_space(3))) uint32_t* LdsWords;
  const int64_t tok_stride = (int64_t)KVH * HD;
  const kv16_t* const kbase = (const kv16_t*)kv.k + (int64_t)layer * kv.layer_stride + (int64_t)g * HD;
  const kv16_t* const vbase = (const kv16_t*)kv.v + (int64_t)layer * kv.layer_stride + (int64_t)g * HD;
  auto turn_k = [](int key) { return HD == 128 ? key & 15 : (key >> 1) & 7; };
  auto turn_v = [](int key) { return HD == 128 ? 2 * (key & 7) : 2 * ((key >> 1) & 3); };
  auto request = [&](int n) {  // this wave's share of tile n of the split
    const int* const tt = tokens + (n / TOK_TILES & 1) * (TOK_TILES * RTK) + n % TOK_TILES * RTK;
    unsigned char* const to = ring + (n & 1) * SLOT;
#pragma unroll
    for (int i = 0; i < (GROUPS + RW - 1) / RW; ++i) {
      const int kg = wave + i * RW, key = kg * KPI + lane / CPR;
      if (GROUPS % RW && kg >= GROUPS) break;  // uniform over the wave
      const int64_t at = (int64_t)tt[key] * tok_stride;
      __builtin_amdgcn_global_load_lds((GlobalWords)(kbase + at + ((lane % CPR) ^ turn_k(key)) * 8), (LdsWords)(to + kg * 1024), 16, 0, 0);
      __builtin_amdgcn_global_load_lds((GlobalWords)(vbase + at + ((lane % CPR) ^ turn_v(key)) * 8), (LdsWords)(to + TILE + kg * 1024), 16, 0, 0);
    }
  };
  if (n_my > 0) request(0);

  float m_run[1], m_top[1], l_run[1];  // of row srow: scaled reference maximum, score up to which it stays (the same in the four key groups), sum over the lane's own keys
  attn_floatx4 acc[1][DB];    // O^T: dims db * 16 + sg4 * 4 + i of row srow
  m_run[0] = m_top[0] = -INFINITY;
  l_run[0] = 0.f;
#pragma unroll
  for (int db = 0; db < DB; ++db) acc[0][db] = attn_floatx4{0.f, 0.f, 0.f, 0.f};
  unsigned k_off[KS], v_off[DB];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) k_off[ks] = srow * (HD * 2) + ((ks * 4 + sg4) ^ turn_k(srow)) * 16;
  {
    const int key = sg4 * 4 + (srow >> 2);
#pragma unroll
    for (int db = 0; db < DB; ++db) v_off[db] = TILE + key * (HD * 2) + ((2 * db + ((srow >> 1) & 1)) ^ turn_v(key)) * 16 + (srow & 1) * 8;
  }

#pragma unroll 1
  for (int n = 0; n < n_my; ++n) {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(ROWS_WAIT_ALL);  // this wave's share of the tile has arrived, its reads of the one before are done
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    if (n + 1 < n_my) request(n + 1);
    // the next block of keys: looked up at the start of this one, in LDS two tiles later
    const int blk_next = n / TOK_TILES + 1;
    if (blk_next * TOK_TILES < n_my) {
      if (n % TOK_TILES == 0) look_up(blk_next);
      if (n % TOK_TILES == 2) put(blk_next);
    }
    const int key0 = (split + n * eff) * RTK;
    const unsigned char* const sp = ring + (n & 1) * SLOT;
    if (key0 + RTK > kend) {  // uniform over the workgroup: the last tile; V rows past the end become zeros
      for (int i = t; i < RTK * CPR; i += RW * 64)
        if (key0 + i / CPR >= kend) *(uint4*)(ring + (n & 1) * SLOT + TILE + i * 16) = make_uint4(0, 0, 0, 0);
      __syncthreads();
    }
    if (rowless || key0 >= wend) continue;  // uniform over the wave

    // S^T = K Q^T
    attn_floatx4 s2[1][NB];
#pragma unroll
    for (int blk = 0; blk < NB; ++blk) s2[0][blk] = attn_floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int blk = 0; blk < NB; ++blk) {
        const half8 kf = *(const half8*)(sp + k_off[ks] + blk * (16 * HD * 2));
        s2[0][blk] = __builtin_amdgcn_mfma_f32_16x16x32_f16(kf, qh[0][ks], s2[0][blk], 0, 0, 0);
        s2[0][blk] = __builtin_amdgcn_mfma_f32_16x16x32_f16(kf, ql[0][ks], s2[0][blk], 0, 0, 0);
      }
    half8 ph[1][NB / 2], pl[1][NB / 2];
    attn_softmax<1, NB, DB, CAUSAL>(s2, rmask, m_run, m_top, l_run, acc, ph, pl, scale, key0, len, all, kend, sg4);
    // O^T += V^T P^T
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int hb = 0; hb < NB / 2; ++hb) {
        const half4 v0 = lds_columns((const _Float16*)(sp + v_off[db] + hb * (32 * HD * 2))), v1 = lds_columns((const _Float16*)(sp + v_off[db] + hb * (32 * HD * 2) + 16 * HD * 2));
        const half8 vt = __builtin_shufflevector(v0, v1, 0, 1, 2, 3, 4, 5, 6, 7);
        acc[0][db] = __builtin_amdgcn_mfma_f32_16x16x32_f16(vt, ph[0][hb], acc[0][db], 0, 0, 0);
        acc[0][db] = __builtin_amdgcn_mfma_f32_16x16x32_f16(vt, pl[0][hb], acc[0][db], 0, 0, 0);
      }
  }
  if (rowless) return;
  const int p = wp0 + srow;
  const bool live = p < wp_end;
  const int pc = live ? p : wp0, row = pc % R, head = g * G + pc / R;
  l_run[0] = xsum<32>(xsum<16>(l_run[0]));
  if (eff == 1) {
    const float inv = l_run[0] > 0.f ? 1.0f / l_run[0] : 0.f;
#pragma unroll
    for (int db = 0; db < DB; ++db) {
      const float x[4] = {acc[0][db][0] * inv, acc[0][db][1] * inv, acc[0][db][2] * inv, acc[0][db][3] * inv};
      uint2 hi, lo;
      split_bf16_x4(x, hi, lo);
      const int k = head * HD + db * 16 + sg4 * 4;
      if (live) {
        *(uint2*)(out + act_offset(ncg, B * R, n_heads * HD, 0, seq * R + row, k)) = hi;
        *(uint2*)(out + act_offset(ncg, B * R, n_heads * HD, 1, seq * R + row, k)) = lo;
      }
    }
  } else if (live) {
    float* const pp = partial + ((((int64_t)seq * n_heads + head) * R + row) * n_splits + split) * (HD + 2);
#pragma unroll
    for (int db = 0; db < DB; ++db) {
      *(float2*)(pp + 2 + db * 16 + sg4 * 4) = make_float2(acc[0][db][0], acc[0][db][1]);
      *(float2*)(pp + 2 + db * 16 + sg4 * 4 + 2) = make_float2(acc[0][db][2], acc[0][db][3]);
    }
    if (sg4 == 0) *(float2*)pp = make_float2(m_run[0], l_run[0]);
  }
}

// Merge of the key splits, a kernel of its own: one wave per (sequence, query head, row).  As a separate launch it is
// spread over the whole machine and costs about the same for any number of
// splits, where the last workgroup of an item merging inside the attention kernel (the first design: 3.3 us of 13.1 at
// 4 splits and 5 rows, 8 us of 28 at 8 splits and 17 rows) made more splits cost more than they gained.
template <int HD>
__global__ __launch_bounds__(256) void attn_merge_kernel(RowDesc rd, KvView kv, int B, int R, int n_heads, const float* __restrict__ partial,
                                                         int n_splits, int want_splits, bf16_t* __restrict__ out, int ncg, bool causal) {
  const int lane = threadIdx.x & 63;
  const int item = blockIdx.x * 4 + (threadIdx.x >> 6);  // (seq, head, row)
  if (item >= B * n_heads * R) return;
  const int row = item % R, head = (item / R) % n_heads, seq = item / (R * n_heads);
  const int eff = attn_splits(attn_keys(kv, rd, seq, causal), n_splits, want_splits);
  if (eff == 1) return;  // the attention kernel wrote the output itself
  const float* pp = partial + (((int64_t)seq * n_heads + head) * R + row) * n_splits * (HD + 2);
  attn_merge_row<HD, false>(pp, eff, out, ncg, B * R, n_heads * HD, seq * R + row, head, lane);
}

// Key splits for `items` workgroups per split: enough workgroups to fill the machine once (twice and four times over measured no faster
// at 512, 2048 and 4096 keys when once is an even fill).  An uneven fill (160 items x 2 splits on 256 compute units) runs as long as the
// compute units that hold two workgroups: then the splits with which a compute unit of n = 2 .. per_cu workgroups holds the least of an item,
// n / splits; two workgroups get a tenth more done together than three or four.  us of a pass of four narrow layers (4 sequences) with the
// splits of 2 / 3 / 4 workgroups: 40 heads x 41 rows x 128 (160 items) 3 / 4 splits, 2064 keys 381 / 398, 4100 keys 517 / 531; 48 heads x 33 rows x
// 128 2 / 4 / 5 splits, 4100 keys 587 / 567 / 583; 24 heads x 57 rows x 128 5 / 8, 4100 keys 403 / 426; one row x 40 heads x 64, 2 sequences, 6 / 9 / 12,
// 4100 keys 179 / 185 / 182, 8 sequences 1 / 2 / 3, 2064 keys 286 / 267 / 256.
// least_keys: from how many keys on a sequence is split.
int splits_wanted(int items, int per_cu, int least_keys) {
  const int n_cus = device_cus(), fill = items >= n_cus ? 1 : (n_cus + items - 1) / items;
  int more = 0;
  float least = INFINITY;
  for (int n = 2; items * fill > n_cus && n <= per_cu; ++n) {
    const int splits = n_cus * n / items;
    const float share = (n == 2 ? 0.9f : 1.f) * n / splits;
    if (splits > 0 && share < least) least = share, more = splits;
  }
  return (fill < 255 ? fill : 255) | (more < 255 ? more : 255) << 8 | least_keys / ATK << 16;
}
// Most workgroups a compute unit.  Items of one or two row groups: those that are resident, but 4 for head dim 64 and one row group (3
// resident; 8 sequences above).  Items of many rows: 3; up to 5 are resident, and no faster (5 x 41 rows x 40 heads x 128, 2064 keys, 2 / 3 / 4
// workgroups 422 / 424 / 453; 4 x 33 rows x 48 heads x 64, 4100 keys 405 / 374 / 386).
constexpr int item_per_cu(int hd, int nrg) { return hd == 64 && nrg == 1 ? 4 : 2; }
constexpr int ROWS_PER_CU = 3;
// Keys from which on items of many rows are split where they give at least every other compute unit a workgroup: below, the merge's launch
// costs more than the tiles it saves a workgroup (14 of 32 keys, 10 of 64).  us of a pass of four narrow layers, split / whole: 32 x 8 rows x 32 heads on 4 x 128,
// 300, 400, 516 keys 255 / 235, 250 / 243, 255 / 266; 4 x 33 rows x 40 heads x 128, 300, 400, 516 keys 262 / 262, 267 / 272, 276 / 293; 8 x 29 rows x 32
// heads on 8 x 64, 300, 516 keys 227 / 212, 233 / 228; 4 x 33 rows x 32 heads x 64, 700 keys 230 / 243; prompts of 300 tokens x 32 heads x 128 226 / 217.
// A prompt's rows see half of its keys on average and are many to merge (split / whole in a launch that offers splits): 31 heads x 128, 479 tokens 261 / 240,
// 20 heads 220 / 215, 16 heads, 600 tokens 222 / 229; 12 heads x 64, 700 tokens 193 / 189, 8 heads, 1000 tokens 189 / 192.
int rows_least_keys(int hd, int items, bool causal) { return 2 * items < device_cus() ? 0 : hd == 128 ? (causal ? 544 : 448) : (causal ? 960 : 640); }
int widest_split(int n_splits, int want) {
  const int fill = want & 255, more = want >> 8 & 255, widest = fill > more ? fill : more;
  return n_splits < widest ? n_splits : widest;
}

template <int HD>
hipError_t run_merge(const RowDesc& rd, const KvView& kv, int B, int R, int n_heads, const float* partial, int n_splits, int want, void* out, int ncg, bool causal,
                    hipStream_t s) {
  hipLaunchKernelGGL((attn_merge_kernel<HD>), dim3((B * n_heads * R + 3) / 4), dim3(256), 0, s, rd, kv, B, R, n_heads, partial, n_splits, want, (bf16_t*)out, ncg,
                     causal);
  return hipGetLastError();
}

template <int HD, int RW, bool CAUSAL>
hipError_t run_rows(const float* q, int q_stride, const RowDesc& rd, const KvView& kv, int layer, int B, int R, int n_heads, float* partial, int n_splits,
                    void* out, int ncg, hipStream_t s) {
  using Sh = RowsShape<HD, RW>;
  const int KVH = kv.n_kv_heads, G = n_heads / KVH, n_chunks = (G * R + RW * 16 - 1) / (RW * 16), items = KVH * n_chunks * B;
  auto kern = tree_attn_rows_kernel<HD, RW, CAUSAL>;
  static_assert(Sh::LDS <= 64 * 1024, "needs no attribute");
  const int want = splits_wanted(items, ROWS_PER_CU, rows_least_keys(HD, items, CAUSAL)), gx = widest_split(n_splits, want);
  const bool spread = spread_splits(gx, items);
  hipLaunchKernelGGL(kern, rows_grid(spread, gx, items), dim3(RW * 64), Sh::LDS, s, q, q_stride, rd, kv, layer, B, R, n_heads, n_chunks,
                     ATTN_LOG2E / sqrtf((float)HD), partial, n_splits, (bf16_t*)out, want, ncg, spread ? 0 : gx);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess || gx == 1) return e;  // one split: every workgroup wrote its output
  return run_merge<HD>(rd, kv, B, R, n_heads, partial, n_splits, want, out, ncg, CAUSAL, s);
}

template <int HD, int NRG, int AW>
hipError_t run_mfma(const float* q, int q_stride, const RowDesc& rd, const KvView& kv, int layer, int B, int R, int n_heads, float* partial,
                    int n_splits, void* out, int ncg, hipStream_t s, int* counters = nullptr) {
  const int KVH = kv.n_kv_heads, G = n_heads / KVH;
  if (G * R > NRG * 16) return hipErrorInvalidValue;  // one item a KV head
  const float scale = ATTN_LOG2E / sqrtf((float)HD);
  auto kern = tree_attn_mfma_kernel<HD, NRG, AW>;
  constexpr size_t lds = sizeof(MfmaAttnSmem<HD, NRG, AW>);
  static const hipError_t attr = lds > 64 * 1024 ? hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds)
                                                 : hipSuccess;
  if (attr != hipSuccess) return attr;
  const int items = KVH * B;
  const int want = splits_wanted(items, item_per_cu(HD, NRG), 0), gx = widest_split(n_splits, want);
  const bool spread = spread_splits(gx, items);
  if constexpr (NRG == 1) {
    // Six layers, us, two launches / one (rows = sequences x heads x rows each): 12 heads x 64, 12 rows, 256 / 2048 keys 164 / 153,
    // 179 / 171; 48 rows 170 / 159, 216 / 208; 32 heads x 64, 64 rows 218 / 198, 241 / 234.  Beyond, the last workgroups' merges
    // are no longer hidden: 96 rows, 2048 keys 252 / 261; 512 rows 292 / 315, 584 / 618.  Items of 8 rows (8 query heads on a key
    // head), two to a wave and few items to split the keys over: 2048 keys 204 / 211.
    if (counters && gx > 1 && B * n_heads * R <= FEW_ROWS && G * R <= ATTN_WAVES) {
      hipLaunchKernelGGL((tree_attn_few_kernel<HD>), attn_grid(spread, gx, KVH, B), dim3(AW * 64), 0, s, q, q_stride, rd, kv, layer, B, R, n_heads, scale,
                         partial, n_splits, (bf16_t*)out, want, ncg, spread, counters);
      return hipGetLastError();
    }
  }
  hipLaunchKernelGGL(kern, attn_grid(spread, gx, KVH, B), dim3(AW * 64), lds, s, q, q_stride, rd, kv, layer, B, R, n_heads, scale, partial, n_splits,
                     (bf16_t*)out, want, ncg, spread);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || gx == 1) return e;  // one split: every workgroup wrote its output
  return run_merge<HD>(rd, kv, B, R, n_heads, partial, n_splits, want, out, ncg, false, s);
}

}  // namespace


// bf16 models: q float32 [B*R][q_stride], half-precision cache, output = bf16 hi / lo planes [2][B*R][n_heads*hd].
// Items of 16 or 32 (query head, row) pairs on a KV head with key tiles dealt to the waves; with more pairs the waves share the tiles
// (both sides of the line: tree_attn_rows_kernel).
hipError_t launch_attention_mfma(const float* q, int q_stride, const RowDesc& rd, KvView kv, int layer, int B, int R, int n_heads,
                                 float* partial, int n_splits, void* out, int ncg, hipStream_t s, int* counters) {
  const int hd = kv.head_dim;
  if (kv.n_kv_heads < 1 || n_heads % kv.n_kv_heads) return hipErrorInvalidValue;
  const int pairs = n_heads / kv.n_kv_heads * R;  // (query head, row) pairs that share a KV head
  if (hd == 128 && pairs <= 16) return run_mfma<128, 1, 4>(q, q_stride, rd, kv, layer, B, R, n_heads, partial, n_splits, out, ncg, s, counters);
  if (hd == 128 && pairs <= 32) return run_mfma<128, 2, 4>(q, q_stride, rd, kv, layer, B, R, n_heads, partial, n_splits, out, ncg, s);
  if (hd == 128 && pairs <= 48) return run_rows<128, 3, false>(q, q_stride, rd, kv, layer, B, R, n_heads, partial, n_splits, out, ncg, s);
  if (hd == 128) return run_rows<128, 4, false>(q, q_stride, rd, kv, layer, B, R, n_heads, partial, n_splits, out, ncg, s);
  if (hd == 64 && pairs <= 16) return run_mfma<64, 1, 4>(q, q_stride, rd, kv, layer, B, R, n_heads, partial, n_splits, out, ncg, s, counters);
  if (hd == 64 && pairs <= 32) return run_mfma<64, 2, 4>(q, q_stride, rd, kv, layer, B, R, n_heads, partial, n_splits, out, ncg, s);
  if (hd == 64 && pairs <= 48) return run_rows<64, 3, false>(q, q_stride, rd, kv, layer, B, R, n_heads, partial, n_splits, out, ncg, s);
  if (hd == 64) return run_rows<64, 4, false>(q, q_stride, rd, kv, layer, B, R, n_heads, partial, n_splits, out, ncg, s);
  return hipErrorInvalidValue;
}

// the rows of a prompt chunk (any number per sequence; causal)
hipError_t launch_attention_prompt(const float* q, int q_stride, const RowDesc& rd, KvView kv, int layer, int B, int R, int n_heads, float* partial,
                                   int n_splits, void* out, int ncg, hipStream_t s) {
  if (kv.n_kv_heads < 1 || n_heads % kv.n_kv_heads) return hipErrorInvalidValue;
  if (kv.head_dim == 128) return run_rows<128, 4, true>(q, q_stride, rd, kv, layer, B, R, n_heads, partial, n_splits, out, ncg, s);
  if (kv.head_dim == 64) return run_rows<64, 4, true>(q, q_stride, rd, kv, layer, B, R, n_heads, partial, n_splits, out, ncg, s);
  return hipErrorInvalidValue;
}

}  // namespace mtad

// Host side only, for the tests: the (split, KV head, sequence, chunk of rows) of every workgroup of an attention launch, in the order they are
// dispatched; at: 4 ints each.
extern "C" void mtad_test_attention_places(int rows, int n_kv_heads, int chunks, int batch, int offered, int spread, int* at) {
  using namespace mtad;
  const int items = n_kv_heads * batch * chunks;
  const dim3 g = rows ? rows_grid(spread != 0, offered, items) : attn_grid(spread != 0, offered, n_kv_heads, batch);
  for (unsigned z = 0; z < g.z; ++z)
    for (unsigned y = 0; y < g.y; ++y)
      for (unsigned x = 0; x < g.x; ++x, at += 4) {
        const AttnPlace p = rows ? rows_place(spread ? 0 : offered, n_kv_heads, batch, x, y) : attn_place(spread != 0, n_kv_heads, x, y, z);
        at[0] = p.split, at[1] = p.g, at[2] = p.seq, at[3] = p.chunk;
      }
}
// Host side only, for the tests: the key splits a launch offers (out[0]) and a sequence of `keys` keys uses (out[1]), and the launch's items
// (out[2]), for `pairs` (query head, row) pairs on a KV head.  They hold for 256 compute units where there is no device.
extern "C" void mtad_test_attention_splits(int head_dim, int pairs, int n_kv_heads, int batch, int causal, int n_splits, int keys, int* out) {
  using namespace mtad;
  const bool rows = causal || pairs > 32, four = causal || pairs > 48;
  const int items = n_kv_heads * batch * (rows ? (pairs + (four ? 63 : 47)) / (four ? 64 : 48) : 1);
  const int want = rows ? splits_wanted(items, ROWS_PER_CU, rows_least_keys(head_dim, items, causal != 0)) : splits_wanted(items, item_per_cu(head_dim, pairs > 16 ? 2 : 1), 0);
  out[0] = widest_split(n_splits, want);
  out[1] = attn_splits(keys, out[0], want);
  out[2] = items;
}
