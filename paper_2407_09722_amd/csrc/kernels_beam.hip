// Integer / decision side of one MTAD iteration: row descriptors of the draft and target passes, the
// beam top-b over beam x vocab candidates (Section 2.1, Eq. 2), the tree of the target pass (Section
// 3.3), the gather of the draft tokens' log-likelihoods, joint-likelihood acceptance with the bonus
// token (Algorithm 1; Eq. 9) and the KV commit / rollback.
#include "common.h"
#include "beam.h"

namespace mtad {

// ---- counter-based noise: SplitMix64 finaliser keyed by (seed, stream, position, index) ------------
__device__ __forceinline__ uint64_t mix64(uint64_t z) {
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}
constexpr uint64_t GOLDEN = 0x9E3779B97F4A7C15ull;
__device__ __forceinline__ uint64_t noise_key(uint64_t seed, int stream, int position) {
  return mix64(mix64(seed ^ (GOLDEN * (uint64_t)(stream + 1))) + (uint64_t)position);
}
// standard Gumbel from the top 23 hash bits: u = (k + 1/2) / 2^23 is exact in float32
__device__ __forceinline__ float gumbel(uint64_t key, uint64_t idx) {
  const uint64_t h = mix64(key ^ (GOLDEN * (idx + 1)));
  const float u = ((float)(uint32_t)(h >> 41) + 0.5f) * 1.1920928955078125e-07f;
  return -logf(-logf(u));
}
constexpr int STREAM_BONUS = 0, STREAM_BEAM = 1, STREAM_ACCEPT = 2, STREAMS_PER_SEQ = 4;
// the uniform number behind the noise: u = (k + 1/2) / 2^23, exact in float32
__device__ __forceinline__ float uniform01(uint64_t key, uint64_t idx) {
  const uint64_t h = mix64(key ^ (GOLDEN * (idx + 1)));
  return ((float)(uint32_t)(h >> 41) + 0.5f) * 1.1920928955078125e-07f;
}

// ---- row descriptors ------------------------------------------------------------------------------

// chain mask: bits 0..r
__device__ __forceinline__ uint64_t chain_bits(int r) { return (r >= 63) ? ~0ull : ((1ull << (r + 1)) - 1ull); }

__device__ __forceinline__ void draft_row(const RowDesc& rd, const int32_t* __restrict__ len, const BeamView& hist, const int32_t* __restrict__ cu_tok,
                                          const int32_t* __restrict__ cu_cnt, int step, int B, int R, int gamma, int beam, int cap,
                                          uint32_t* __restrict__ status) {
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= B * R) return;
  const int s = idx / R, r = idx % R;
  int cnt = cu_cnt[s];
  if (cnt < 1 || cnt > gamma + 1) {
    if (r == 0) atomicOr(status, (uint32_t)ST_BAD_CATCHUP);
    cnt = 1;
  }
  const int n = len[s];
  int tok = 0, pos = 0, slot = -1;
  uint64_t mask = 0;
  if (step == 0) {
    if (r < cnt) {
      tok = cu_tok[s * (gamma + 1) + r];
      pos = n + r;
      slot = n + r;
      mask = chain_bits(r);
    }
    if (r == 0) rd.nspec[s] = cnt;
  } else {
    const int rel = cnt + (step - 1) * beam + r;
    if (rel < 64) {
      tok = hist.tok[(s * gamma + step - 1) * beam + r];
      pos = n + cnt - 1 + step;
      slot = n + rel;
      mask = chain_bits(cnt - 1) | (1ull << rel);
      int jj = r;
      for (int ii = step - 1; ii >= 1; --ii) {  // ancestors fed at steps ii = step-1 .. 1
        jj = min(max(hist.parent[(s * gamma + ii) * beam + jj], 0), beam - 1);  // caller-owned memory: stay in range
        mask |= 1ull << (cnt + (ii - 1) * beam + jj);
      }
    } else if (r == 0) {
      atomicOr(status, (uint32_t)ST_SPEC_WINDOW);
    }
    if (r == 0) rd.nspec[s] = min(64, cnt + step * beam);
  }
  if (slot >= cap) {
    atomicOr(status, (uint32_t)ST_KV_CAP);
    slot = -1;
  }
  rd.tok[idx] = tok;
  rd.pos[idx] = pos;
  rd.slot[idx] = slot;
  rd.mask[idx] = mask;
}

__global__ void draft_rows_kernel(RowDesc rd, const int32_t* __restrict__ len, BeamView hist, const int32_t* __restrict__ cu_tok,
                                  const int32_t* __restrict__ cu_cnt, int step, int B, int R, int gamma, int beam, int cap,
                                  uint32_t* __restrict__ status, PassCount count) {
  const uint32_t last = last_pass(count);
  draft_row(rd, len, hist, cu_tok, cu_cnt, step, B, R, gamma, beam, cap, status);
  if (blockIdx.x == 0) count_pass(count, last, threadIdx.x);
}

hipError_t launch_draft_rows(const RowDesc& rd, const int32_t* len, BeamView hist, const int32_t* cu_tok, const int32_t* cu_cnt,
                             int step, int B, int R, int gamma, int beam, int cap, uint32_t* status, const PassCount& count, hipStream_t s) {
  hipLaunchKernelGGL(draft_rows_kernel, dim3((B * R + 63) / 64), dim3(64), 0, s, rd, len, hist, cu_tok, cu_cnt, step, B, R, gamma,
                     beam, cap, status, count);
  return hipGetLastError();
}

__device__ __forceinline__ void verify_row(const RowDesc& rd, const int32_t* __restrict__ len, const int32_t* __restrict__ root_tok, const TreeView& tree,
                                           int B, int cap, uint32_t* __restrict__ status) {
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  const int M = tree.M;
  if (idx >= B * M) return;
  const int s = idx / M, r = idx % M;
  const int n = len[s];
  int slot = n + r;
  if (slot >= cap) {
    atomicOr(status, (uint32_t)ST_KV_CAP);
    slot = -1;
  }
  rd.tok[idx] = (r == 0) ? root_tok[s] : tree.tok[idx];
  rd.pos[idx] = n + tree.depth[idx];
  rd.slot[idx] = slot;
  rd.mask[idx] = tree.anc_mask[idx];
  if (r == 0) rd.nspec[s] = M;
}

__global__ void verify_rows_kernel(RowDesc rd, const int32_t* __restrict__ len, const int32_t* __restrict__ root_tok, TreeView tree,
                                   int B, int cap, uint32_t* __restrict__ status, PassCount count) {
  const uint32_t last = last_pass(count);
  verify_row(rd, len, root_tok, tree, B, cap, status);
  if (blockIdx.x == 0) count_pass(count, last, threadIdx.x);
}

hipError_t launch_verify_rows(const RowDesc& rd, const int32_t* len, const int32_t* root_tok, TreeView tree, int B, int cap,
                              uint32_t* status, const PassCount& count, hipStream_t s) {
  hipLaunchKernelGGL(verify_rows_kernel, dim3((B * tree.M + 63) / 64), dim3(64), 0, s, rd, len, root_tok, tree, B, cap, status, count);
  return hipGetLastError();
}

// causal chunk of a prompt: rows c0 .. c0+R-1 of tokens[B][n]
__global__ void prefill_rows_kernel(RowDesc rd, const int32_t* __restrict__ len, const int32_t* __restrict__ tokens, int n, int c0,
                                    int B, int R, int cap, uint32_t* __restrict__ status) {
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= B * R) return;
  const int s = idx / R, r = idx % R;
  const int base = len[s];
  int tok = 0, pos = 0, slot = -1;
  uint64_t mask = 0;
  if (c0 + r < n) {
    tok = tokens[(int64_t)s * n + c0 + r];
    pos = base + r;
    slot = base + r;
    mask = chain_bits(r);
    if (slot >= cap) {
      atomicOr(status, (uint32_t)ST_KV_CAP);
      slot = -1;
    }
  }
  rd.tok[idx] = tok;
  rd.pos[idx] = pos;
  rd.slot[idx] = slot;
  rd.mask[idx] = mask;
  if (r == 0) rd.nspec[s] = min(R, n - c0);
}

__global__ void advance_len_kernel(int32_t* len, const int32_t* __restrict__ nspec, int B, int cap) {
  const int s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s < B) len[s] = min(cap, len[s] + nspec[s]);
}

hipError_t launch_prefill_rows(const RowDesc& rd, const int32_t* len, const int32_t* tokens, int n, int c0, int B, int R, int cap,
                               uint32_t* status, hipStream_t s) {
  hipLaunchKernelGGL(prefill_rows_kernel, dim3((B * R + 63) / 64), dim3(64), 0, s, rd, len, tokens, n, c0, B, R, cap, status);
  return hipGetLastError();
}
hipError_t launch_advance_len(int32_t* len, const int32_t* nspec, int B, int cap, hipStream_t s) {
  hipLaunchKernelGGL(advance_len_kernel, dim3((B + 63) / 64), dim3(64), 0, s, len, nspec, B, cap);
  return hipGetLastError();
}

// ---- beam top-b -----------------------------------------------------------------------------------

constexpr int MAXB = 8;

__device__ __forceinline__ bool better(float k1, int i1, float k2, int i2) { return k1 > k2 || (k1 == k2 && i1 < i2); }

// (key, idx) as one unsigned number that is larger exactly where better() says so: the key's bits in an order that compares as
// unsigned (both zeros alike; no NaN), then the complement of idx.
__device__ __forceinline__ uint64_t rank_of(float k, int i) {
  const uint32_t u = __float_as_uint(k + 0.0f);  // -0 becomes +0
  return ((uint64_t)(u ^ ((u >> 31) ? 0xFFFFFFFFu : 0x80000000u)) << 32) | (uint32_t)~i;
}
__device__ __forceinline__ float rank_key(uint64_t r) {
  const uint32_t u = (uint32_t)(r >> 32);
  return __uint_as_float(u ^ ((u >> 31) ? 0x80000000u : 0xFFFFFFFFu));
}
__device__ __forceinline__ int rank_idx(uint64_t r) { return (int)~(uint32_t)r; }

// one step of a maximum over lanes: the value CTRL's lane pattern brings, where ROWS lets it in
template <int CTRL, int ROWS>
__device__ __forceinline__ uint64_t max_step(uint64_t v) {
  const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp((int)(v >> 32), (int)(v >> 32), CTRL, ROWS, 0xf, false);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp((int)(uint32_t)v, (int)(uint32_t)v, CTRL, ROWS, 0xf, false);
  const uint64_t o = ((uint64_t)hi << 32) | lo;
  return o > v ? o : v;
}
template <int LANE>
__device__ __forceinline__ uint64_t from_lane(uint64_t v) {
  return ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(v >> 32), LANE) << 32) | (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, LANE);
}
// largest value of lanes 0 .. 15, and of the whole wave, in every lane: data-parallel-primitive moves in the vector ALU, a
// dozen clocks a step where a shuffle through LDS takes over a hundred
__device__ __forceinline__ uint64_t row_max(uint64_t v) {
  v = max_step<0x111, 0xf>(v);  // row_shr:1, 2, 4, 8: lane 15 of a row of 16 has the row's maximum
  v = max_step<0x112, 0xf>(v);
  v = max_step<0x114, 0xf>(v);
  v = max_step<0x118, 0xf>(v);
  return from_lane<15>(v);
}
__device__ __forceinline__ uint64_t wave_max_rank(uint64_t v) {
  v = max_step<0x111, 0xf>(v);
  v = max_step<0x112, 0xf>(v);
  v = max_step<0x114, 0xf>(v);
  v = max_step<0x118, 0xf>(v);
  v = max_step<0x142, 0xa>(v);  // row_bcast:15 into rows 1 and 3, row_bcast:31 into rows 2 and 3
  v = max_step<0x143, 0xc>(v);
  return from_lane<63>(v);
}
// of a workgroup of at most 16 waves; sh: 16 entries.  One barrier; the caller may use sh again only after another one.
__device__ __forceinline__ uint64_t block_max_rank(uint64_t v, uint64_t* sh) {
  v = wave_max_rank(v);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  const int nw = (int)blockDim.x >> 6;
  return row_max(sh[min((int)(threadIdx.x & 15), nw - 1)]);
}

// The b best (b <= 8) of the entries the lanes of a wave hold, N each, and of `kept` (what an earlier call left): lane j < b gets
// the j-th best, the others the empty entry.  b rounds over the lanes' best entries give a threshold; what reaches it (in at
// most b lanes) is listed in LDS, and b more rounds pick from the list.  No lane searches its entries more than twice.
// list: TOP_LIST entries of the wave's own.
constexpr uint64_t NO_RANK = ((uint64_t)0x007FFFFFu << 32) | 0x80000000u;  // rank_of(-infinity, 0x7FFFFFFF)
constexpr int TOP_N = 16, TOP_LIST = MAXB * (TOP_N + 1);
template <int N, bool ONE = false>
__device__ __forceinline__ uint64_t wave_top(const uint64_t (&e)[N], uint64_t kept, int b, uint64_t* list, int* count) {
  static_assert(N <= TOP_N, "list size");
  const int lane = threadIdx.x & 63;
  uint64_t mine = kept;
#pragma unroll
  for (int j = 0; j < N; ++j) mine = e[j] > mine ? e[j] : mine;
  if constexpr (ONE) return wave_max_rank(mine);  // b = 1: nothing to list
  uint64_t left = mine, T = 0;
  for (int r = 0; r < b; ++r) {
    T = wave_max_rank(left);
    if (left == T) left = 0;
  }
  T = T > NO_RANK ? T : NO_RANK + 1;  // empty entries are not listed
  if (lane == 0) *count = 0;
  __builtin_amdgcn_wave_barrier();
  if (mine >= T) {
    if (kept >= T) list[atomicAdd(count, 1)] = kept;
#pragma unroll
    for (int j = 0; j < N; ++j)
      if (e[j] >= T) list[atomicAdd(count, 1)] = e[j];
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  const int n = *(volatile int*)count;
  constexpr int P = (TOP_LIST + 63) / 64;
  uint64_t c[P], top = NO_RANK;
#pragma unroll
  for (int p = 0; p < P; ++p) c[p] = lane + 64 * p < n ? ((volatile uint64_t*)list)[lane + 64 * p] : NO_RANK;
  for (int r = 0; r < b; ++r) {
    uint64_t m = c[0];
#pragma unroll
    for (int p = 1; p < P; ++p) m = c[p] > m ? c[p] : m;
    m = wave_max_rank(m);
    if (lane == r) top = m;
#pragma unroll
    for (int p = 0; p < P; ++p)
      if (c[p] == m) c[p] = NO_RANK;
  }
  return top;
}
struct TopShared {
  uint64_t list[4][TOP_LIST], best[4 * MAXB];
  int count[4];
};
// the b best of a workgroup of 256 threads whose waves hold theirs as wave_top leaves them: lane j < b of wave 0 gets the j-th
__device__ __forceinline__ uint64_t block_top(uint64_t top, int b, TopShared& sh) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane < MAXB) sh.best[wave * MAXB + lane] = lane < b ? top : NO_RANK;
  __syncthreads();
  if (wave == 0) {
    uint64_t v = lane < 4 * MAXB ? sh.best[lane] : NO_RANK;
    for (int j = 0; j < b; ++j) {
      const uint64_t m = wave_max_rank(v);
      if (v == m) v = NO_RANK;
      if (lane == j) top = m;
    }
  }
  return top;
}

// score of candidate (live beam r, token v): cum_logq[r] + (logit - lse), float32, in this order
__device__ __forceinline__ float cand_score(const float* logits, const float* lse, const float* cum, int row0, int r, int v, int V) {
  const int row = row0 + r;
  return cum[r] + (logits[(int64_t)row * V + v] - lse[row]);
}

// stage 1: grid (G, B); block g scans its slice of the n_live*V candidates, N per thread at a time.  ONE: one survivor.
template <int N, bool ONE>
__global__ __launch_bounds__(256) void topb_stage1_kernel(const float* __restrict__ logits, const float* __restrict__ lse, BeamView hist,
                                                          const int32_t* __restrict__ cu_cnt, const int32_t* __restrict__ len, int step,
                                                          int R, int gamma, int beam, int V, int sample, uint64_t seed,
                                                          float* __restrict__ part_key, int* __restrict__ part_idx,
                                                          const float2* __restrict__ lse_part, int NP, float* __restrict__ lse_out) {
  __shared__ TopShared sh;
  __shared__ float lse_sh[4], lse_s[MAXB];
  __shared__ float cum_s[MAXB];
  const int s = blockIdx.y, G = gridDim.x;
  const int n_live = (step == 0) ? 1 : beam;
  int cnt = cu_cnt[s];
  if (cnt < 1 || cnt > gamma + 1) cnt = 1;
  const int row0 = s * R + ((step == 0) ? cnt - 1 : 0);  // step 0: the last catch-up row carries the context distribution
  if (threadIdx.x < MAXB)
    cum_s[threadIdx.x] = (step == 0 || (int)threadIdx.x >= beam) ? 0.f : hist.cum[(s * gamma + step - 1) * beam + threadIdx.x];
  __syncthreads();
  const int total = n_live * V;
  const int per = (total + G - 1) / G;
  const int c0 = blockIdx.x * per, c1 = min(total, c0 + per);
  const uint64_t nk = noise_key(seed, s * STREAMS_PER_SEQ + STREAM_BEAM, len[s] + cnt + step);
  // lse_part: the rows' logsumexps are still partial sums per strip of the lm_head; every workgroup finishes those of its slice
  // (all write the same value) instead of a launch in between
  if (lse_part && c0 < c1)
    for (int r = c0 / V; r <= (c1 - 1) / V; ++r) {
      const float l = lse_of_row(lse_part + (int64_t)(row0 + r) * NP, NP, lse_sh);
      if (threadIdx.x == 0) {
        lse_s[r] = l;
        lse_out[row0 + r] = l;
      }
    }
  __syncthreads();
  // N candidates per thread at a time, their logits requested together.  A slice lies in at most two rows (a workgroup has 1/G of at
  // most MAXB of them, and G >= MAXB): their likelihoods and logsumexps are looked up once, not per candidate behind a division.
  const int ra = min(c0 / V, n_live - 1), rb = min(ra + 1, n_live - 1), rb_at = (ra + 1) * V;
  const float cum_a = cum_s[ra], cum_b = cum_s[rb];
  float lse_a = 0.f, lse_b = 0.f;
  if (c0 < c1) {
    lse_a = lse_part ? lse_s[ra] : lse[row0 + ra];
    if (c1 > rb_at) lse_b = lse_part ? lse_s[rb] : lse[row0 + rb];
  }
  const int wave = threadIdx.x >> 6;
  uint64_t top = NO_RANK;
  for (int cb = c0 + (int)threadIdx.x; cb - (int)threadIdx.x < c1; cb += 256 * N) {
    uint64_t e[N];
    float x[N];
#pragma unroll
    for (int u = 0; u < N; ++u) {
      const int c = min(cb + 256 * u, c1 - 1);
      x[u] = logits[(int64_t)row0 * V + c];  // rows of the live beams follow each other
      x[u] = (c >= rb_at ? cum_b : cum_a) + (x[u] - (c >= rb_at ? lse_b : lse_a));
    }
#pragma unroll
    for (int u = 0; u < N; ++u) {
      const int c = cb + 256 * u;
      e[u] = NO_RANK;
      if (c < c1) {
        if (sample) x[u] += gumbel(nk, (uint64_t)c);
        e[u] = rank_of(x[u] == x[u] ? x[u] : -INFINITY, c);  // a NaN score never wins and never leaves an empty slot behind
      }
    }
    top = wave_top<N, ONE>(e, top, beam, sh.list[wave], &sh.count[wave]);
  }
  top = block_top(top, beam, sh);
  if ((int)threadIdx.x < beam) {
    part_key[(s * G + blockIdx.x) * MAXB + threadIdx.x] = rank_key(top);
    part_idx[(s * G + blockIdx.x) * MAXB + threadIdx.x] = rank_idx(top);
  }
}

// stage 2: grid (B); merge G*beam partial winners, write the survivors of this step, best first
__global__ __launch_bounds__(256) void topb_stage2_kernel(const float* __restrict__ logits, const float* __restrict__ lse, BeamView hist,
                                                          const int32_t* __restrict__ cu_cnt, int step, int R, int gamma, int beam,
                                                          int V, int G, const float* __restrict__ part_key,
                                                          const int* __restrict__ part_idx) {
  __shared__ TopShared sh;
  __shared__ float cum_s[MAXB];
  const int s = blockIdx.x;
  int cnt = cu_cnt[s];
  if (cnt < 1 || cnt > gamma + 1) cnt = 1;
  const int row0 = s * R + ((step == 0) ? cnt - 1 : 0);
  if (threadIdx.x < MAXB)
    cum_s[threadIdx.x] = (step == 0 || (int)threadIdx.x >= beam) ? 0.f : hist.cum[(s * gamma + step - 1) * beam + threadIdx.x];
  const int wave = threadIdx.x >> 6;
  uint64_t top = NO_RANK;
  for (int eb = threadIdx.x; eb - (int)threadIdx.x < G * beam; eb += 512) {
    uint64_t e[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int n = min(eb + 256 * u, G * beam - 1), at = (s * G + n / beam) * MAXB + n % beam;
      const float k = part_key[at];
      const int i = part_idx[at];
      e[u] = eb + 256 * u < G * beam ? rank_of(k, i) : NO_RANK;
    }
    top = wave_top(e, top, beam, sh.list[wave], &sh.count[wave]);
  }
  top = block_top(top, beam, sh);  // (its barrier also covers cum_s)
  if (threadIdx.x < beam) {
    int c = rank_idx(top);
    if (c < 0 || c >= ((step == 0) ? 1 : beam) * V) c = 0;  // only reachable with non-finite logits: stay in bounds
    const int o = (s * gamma + step) * beam + threadIdx.x;
    const int r = c / V, v = c % V;
    hist.tok[o] = v;
    hist.parent[o] = r;
    hist.cum[o] = cand_score(logits, lse, cum_s, row0, r, v, V);  // the stored likelihood carries no noise
  }
}

hipError_t launch_topb(const float* logits, const float* lse, BeamView hist, const int32_t* cu_cnt, const int32_t* len, int step,
                       int B, int R, int gamma, int beam, int V, int sample, uint64_t seed, float* part_key, int* part_idx, int G,
                       hipStream_t s, const float* lse_part, int NP, float* lse_out) {
  // Sixteen candidates a thread keep the memory busy in a long slice; most of a short one's would be the last one again, and a single
  // survivor needs no list.  With sixteen and the list / with four, and without it for one survivor, 64 workgroups a sequence: beam 1,
  // 32000 tokens, 1, 16 and 64 sequences 8.0 / 5.9, 11.6 / 7.2 and 26.4 / 11.8 us; beam 4, 4096 tokens, one sequence 10.9 / 9.4.
  const int per = ((step == 0 ? 1 : beam) * V + G - 1) / G;
  auto stage1 = [&](auto kern) {
    hipLaunchKernelGGL(kern, dim3(G, B), dim3(256), 0, s, logits, lse, hist, cu_cnt, len, step, R, gamma, beam, V, sample, seed, part_key, part_idx,
                       (const float2*)lse_part, NP, lse_out);
  };
  if (per > 4 * 256) {
    if (beam == 1) stage1(topb_stage1_kernel<TOP_N, true>);
    else stage1(topb_stage1_kernel<TOP_N, false>);
  } else {
    if (beam == 1) stage1(topb_stage1_kernel<4, true>);
    else stage1(topb_stage1_kernel<4, false>);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(topb_stage2_kernel, dim3(B), dim3(256), 0, s, logits, lse, hist, cu_cnt, step, R, gamma, beam, V, G, part_key,
                     part_idx);
  return hipGetLastError();
}

// ---- tree of the target pass --------------------------------------------------------------------------

// One wave per sequence: the history goes to LDS once (read by one thread it was a chain of dependent loads), lane 0 traces x**,
// then every lane fills one row and walks its own ancestors.
__global__ __launch_bounds__(64) void build_tree_kernel(BeamView hist, TreeView tree, int B, int gamma, int beam, int mode) {
  __shared__ int par_s[MTAD_MAX_GAMMA * MAXB], tok_s[MTAD_MAX_GAMMA * MAXB];
  __shared__ float cum_s[MTAD_MAX_GAMMA * MAXB];
  __shared__ int beams[MTAD_MAX_GAMMA];
  const int s = blockIdx.x, lane = threadIdx.x, M = tree.M, n = gamma * beam;
  for (int e = lane; e < n; e += 64) {
    tok_s[e] = hist.tok[(int64_t)s * n + e];
    par_s[e] = min(max(hist.parent[(int64_t)s * n + e], 0), beam - 1);  // caller-owned memory: stay in range
    cum_s[e] = hist.cum[(int64_t)s * n + e];
  }
  __syncthreads();
  if (lane == 0) {
    // x**: final beam with the largest stored likelihood (first maximum), traced back through the parents
    int j = 0;
    for (int k = 1; k < beam; ++k)
      if (cum_s[(gamma - 1) * beam + k] > cum_s[(gamma - 1) * beam + j]) j = k;
    for (int i = gamma - 1; i >= 0; --i) {
      beams[i] = j;
      j = par_s[i * beam + j];
    }
  }
  __syncthreads();
  for (int i = lane; i < gamma; i += 64) tree.qref[s * gamma + i] = cum_s[i * beam + beams[i]];
  for (int r = lane; r < M; r += 64) {
    int tok = -1, par = -1, dep = 0, src = -1;
    uint64_t am = 1ull;
    if (r > 0 && mode == 0) {
      const int i = r - 1;
      tok = tok_s[i * beam + beams[i]];
      par = i;
      dep = i + 1;
      src = beams[i];
      am = chain_bits(r);
    } else if (r > 0) {
      const int i = (r - 1) / beam;
      int k = (r - 1) % beam;
      tok = tok_s[i * beam + k];
      src = k;
      dep = i + 1;
      par = (i == 0) ? 0 : 1 + (i - 1) * beam + par_s[i * beam + k];
      for (int ii = i; ii >= 0; --ii) {
        am |= 1ull << (1 + ii * beam + k);
        k = par_s[ii * beam + k];
      }
    }
    const int64_t o = (int64_t)s * M + r;
    tree.tok[o] = tok;
    tree.parent[o] = par;
    tree.depth[o] = dep;
    tree.src_beam[o] = src;
    tree.anc_mask[o] = am;
  }
}

hipError_t launch_build_tree(BeamView hist, TreeView tree, int B, int gamma, int beam, int mode, hipStream_t s) {
  if (gamma > MTAD_MAX_GAMMA || beam > MAXB) return hipErrorInvalidValue;
  hipLaunchKernelGGL(build_tree_kernel, dim3(B), dim3(64), 0, s, hist, tree, B, gamma, beam, mode);
  return hipGetLastError();
}

// ---- gather of the draft tokens' conditional log-likelihoods ----------------------------------------------

__global__ void gather_logp_kernel(const float* __restrict__ logits, const float* __restrict__ lse, TreeView tree, int B, int V,
                                   float* __restrict__ logp_cond) {
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  const int M = tree.M;
  if (idx >= B * M) return;
  const int s = idx / M, c = idx % M;
  float out = 0.f;
  if (c > 0) {
    const int p = tree.parent[idx], t = tree.tok[idx];
    if (p >= 0 && p < M && t >= 0 && t < V) out = logits[((int64_t)s * M + p) * V + t] - lse[s * M + p];
  }
  logp_cond[idx] = out;
}

hipError_t launch_gather_logp(const float* logits, const float* lse, TreeView tree, int B, int V, float* logp_cond, hipStream_t s) {
  hipLaunchKernelGGL(gather_logp_kernel, dim3((B * tree.M + 63) / 64), dim3(64), 0, s, logits, lse, tree, B, V, logp_cond);
  return hipGetLastError();
}

// ---- joint-likelihood acceptance and bonus token -----------------------------------------------------------

// The walk over a sequence's rows: eta and the accepted node.  The rows go to LDS first (from memory every row was a chain of
// dependent loads).  All threads of a workgroup of at least 64 call it; the result is in w.eta, w.node after the barrier that
// ends it.
struct AcceptWalk {
  float joint[MTAD_MAX_ROWS], cond[MTAD_MAX_ROWS], qref[MTAD_MAX_ROWS];
  int par[MTAD_MAX_ROWS], dep[MTAD_MAX_ROWS], tok[MTAD_MAX_ROWS];
  int eta, node;
};
__device__ __forceinline__ void accept_walk(AcceptWalk& w, const TreeView& tree, const float* __restrict__ logp_cond, int s, float log_tau, int mode,
                                            int gamma) {
  const int M = tree.M, t = threadIdx.x;
  if (t < M) {
    const int64_t o = (int64_t)s * M + t;
    w.par[t] = tree.parent[o];
    w.dep[t] = tree.depth[o];
    w.tok[t] = tree.tok[o];
    w.cond[t] = logp_cond[o];
  }
  if (t < gamma) w.qref[t] = tree.qref[s * gamma + t];  // gamma < MTAD_MAX_ROWS: a context's passes hold gamma + 1 rows
  __syncthreads();
  if (t == 0) {
    // log p of every branch: conditionals summed from the first level down (parents precede children)
    w.joint[0] = 0.f;
    int eta = 0, node = 0;
    float best = -INFINITY;
    for (int c = 1; c < M; ++c) {
      const int p = w.par[c];
      const float jp = w.joint[(p >= 0 && p < c) ? p : 0] + w.cond[c];
      w.joint[c] = jp;
      const int i = w.dep[c];
      if (i < 1 || i > gamma) continue;
      const float diff = jp - w.qref[i - 1];
      if (mode == 0) {
        if (fminf(0.f, diff) > log_tau && i >= eta) { eta = i; node = c; }  // rows of a chain come in depth order
      } else {
        if (diff >= log_tau && (i > eta || (i == eta && jp > best))) { eta = i; node = c; best = jp; }
      }
    }
    w.eta = eta;
    w.node = node;
  }
  __syncthreads();
}
// what the walk alone decides (one thread)
__device__ __forceinline__ void accept_store(const AcceptWalk& w, const AcceptView& out, int s, int M, int gamma) {
  out.eta[s] = w.eta;
  out.bonus_row[s] = w.node;
  out.out_cnt[s] = w.eta + 1;
  for (int i = 0; i < gamma; ++i) out.path[s * gamma + i] = -1;
  int c = w.node;
  for (int i = w.eta; i >= 1 && c > 0 && c < M; --i) {
    out.path[s * gamma + i - 1] = c;
    out.out_tok[s * (gamma + 1) + i - 1] = w.tok[c];
    c = w.par[c];
  }
}
// best entry of v = first, first + step, ... of a (noisy) logits row, eight loads in flight
__device__ __forceinline__ uint64_t best_of_row(const float* __restrict__ row, int V, int first, int step, int sample, uint64_t nk) {
  float bk = -INFINITY;
  int bi = 0x7FFFFFFF;
  constexpr int U = 8;
  for (int vb = first; vb < V; vb += step * U) {
    float k[U];
#pragma unroll
    for (int u = 0; u < U; ++u) k[u] = row[min(vb + step * u, V - 1)];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int v = vb + step * u;
      if (v >= V) continue;
      if (sample) k[u] += gumbel(nk, (uint64_t)v);
      if (better(k[u], v, bk, bi)) { bk = k[u]; bi = v; }  // (never with a NaN)
    }
  }
  return rank_of(bk, bi);
}

// Acceptance and bonus token by one workgroup per sequence (part == null), or, with 2 x gridDim.x words of workspace per
// sequence at `part`, the bonus token's argmax by gridDim.x workgroups: 32000 Gumbel keys are 11 us of one compute unit's arithmetic and
// 1 us of sixteen's.  counters: a zeroed word per sequence, left zeroed, or null (a launch of its own then takes the best of all).
__global__ __launch_bounds__(1024) void accept_kernel(TreeView tree, const float* __restrict__ logp_cond, const float* __restrict__ logits,
                                                     int V, const int32_t* __restrict__ len, float log_tau, int mode, int gamma,
                                                     int sample, uint64_t seed, AcceptView out, uint64_t* __restrict__ part, int* __restrict__ counters) {
  __shared__ AcceptWalk w;
  __shared__ uint64_t sh[16];
  const int s = blockIdx.y, M = tree.M;
  accept_walk(w, tree, logp_cond, s, log_tau, mode, gamma);
  if (blockIdx.x == 0 && threadIdx.x == 0) accept_store(w, out, s, M, gamma);
  const float* row = logits + ((int64_t)s * M + w.node) * V;
  const uint64_t nk = noise_key(seed, s * STREAMS_PER_SEQ + STREAM_BONUS, len[s] + 1 + w.eta);
  uint64_t best = block_max_rank(best_of_row(row, V, blockIdx.x * blockDim.x + threadIdx.x, gridDim.x * blockDim.x, sample, nk), sh);
  if (threadIdx.x >= 64) return;
  if (part) {
    const int G = gridDim.x;
    if (!counters) {  // accept_finish_kernel takes the best of all
      if (threadIdx.x == 0) part[s * G + blockIdx.x] = best;
      return;
    }
    // wave 0 of the workgroup that arrives last takes it
    int prev = 0;
    if (threadIdx.x == 0) {
      __hip_atomic_store((unsigned long long*)part + s * G + blockIdx.x, (unsigned long long)best, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __builtin_amdgcn_s_waitcnt(0);  // acknowledged
      prev = __hip_atomic_fetch_add(counters + s, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (__builtin_amdgcn_readfirstlane(prev) != G - 1) return;
    if (threadIdx.x == 0) __hip_atomic_store(counters + s, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);  // clean for the next launch
    best = row_max(__hip_atomic_load((unsigned long long*)part + s * G + min((int)(threadIdx.x & 15), G - 1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));  // G <= 16
  }
  if (threadIdx.x != 0) return;
  int bi = rank_idx(best);
  if (bi < 0 || bi >= V) bi = 0;  // only reachable with non-finite logits: stay in the vocabulary
  out.bonus_tok[s] = bi;
  out.out_tok[s * (gamma + 1) + w.eta] = bi;
}

__global__ __launch_bounds__(64) void accept_finish_kernel(const uint64_t* __restrict__ part, int G, int V, int gamma, AcceptView out) {
  const int s = blockIdx.x;
  const uint64_t best = row_max(part[s * G + min((int)(threadIdx.x & 15), G - 1)]);  // G <= 16
  if (threadIdx.x != 0) return;
  int bi = rank_idx(best);
  if (bi < 0 || bi >= V) bi = 0;  // only reachable with non-finite logits: stay in the vocabulary
  out.bonus_tok[s] = bi;
  out.out_tok[s * (gamma + 1) + out.out_cnt[s] - 1] = bi;
}

hipError_t launch_accept(TreeView tree, const float* logp_cond, const float* logits, int V, const int32_t* len, float log_tau, int mode,
                         int B, int gamma, int sample, uint64_t seed, AcceptView out, void* part, int* counters, hipStream_t s) {
  // Sixteen workgroups of 256 threads where their partial results have a place and there is noise to compute.  One workgroup / sixteen,
  // us: 1 sequence of 17 rows, 4096, 6144, 8192 and 32000 tokens 7.7 / 7.8, 8.6 / 7.8, 9.2 / 7.9, 19.0 / 8.8; 64 sequences of 2
  // rows 5.4 / 6.4, 6.1 / 6.7, 6.8 / 6.8, 16.8 / 9.2.
  const bool wide = part && sample && V >= 8192;
  if (!wide) {
    hipLaunchKernelGGL(accept_kernel, dim3(1, B), dim3(1024), 0, s, tree, logp_cond, logits, V, len, log_tau, mode, gamma, sample, seed, out,
                       (uint64_t*)nullptr, (int*)nullptr);
    return hipGetLastError();
  }
  // Two launches / one: 32000 tokens, 1, 4, 16 and 64 sequences 8.8 / 8.4, 13.9 / 13.0, 7.1 / 8.6 and 9.0 / 11.4 us (17, 41, 4 and 2 rows each).
  const bool one_launch = counters && B <= 8;
  hipLaunchKernelGGL(accept_kernel, dim3(ACCEPT_PARTS, B), dim3(256), 0, s, tree, logp_cond, logits, V, len, log_tau, mode, gamma, sample, seed, out,
                     (uint64_t*)part, one_launch ? counters : nullptr);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess || one_launch) return e;
  hipLaunchKernelGGL(accept_finish_kernel, dim3(B), dim3(64), 0, s, (const uint64_t*)part, ACCEPT_PARTS, V, gamma, out);
  return hipGetLastError();
}

// ---- vanilla speculative decoding (Section 2.2), the baseline: token-wise acceptance and the correction token ------------

// log q(. | prefix) of the one live beam of a draft step (beam width 1), kept for the accept step: row r of the step's
// logits (the last catch-up row at step 0, row 0 afterwards) minus its logsumexp.  grid (blocks, B).
__global__ __launch_bounds__(256) void save_logq_row_kernel(const float* __restrict__ logits, const float* __restrict__ lse,
                                                            const int32_t* __restrict__ cu_cnt, int step, int R, int gamma, int V,
                                                            float* __restrict__ qrows) {
  const int s = blockIdx.y;
  int r = 0;
  if (step == 0) {
    int cnt = cu_cnt[s];
    if (cnt < 1 || cnt > gamma + 1) cnt = 1;
    r = cnt - 1;
  }
  const float* row = logits + ((int64_t)s * R + r) * V;
  const float l = lse[s * R + r];
  float* out = qrows + ((int64_t)s * gamma + step) * V;
  for (int v = blockIdx.x * blockDim.x + threadIdx.x; v < V; v += gridDim.x * blockDim.x) out[v] = row[v] - l;
}

hipError_t launch_save_logq_row(const float* logits, const float* lse, const int32_t* cu_cnt, int step, int B, int R, int gamma, int V,
                                float* qrows, hipStream_t s) {
  hipLaunchKernelGGL(save_logq_row_kernel, dim3(8, B), dim3(256), 0, s, logits, lse, cu_cnt, step, R, gamma, V, qrows);
  return hipGetLastError();
}

// One workgroup per sequence.  Thread 0 walks the chain: x_t passes when log u_t < min(0, log p(x_t) - log q(x_t)), u_t
// keyed by the token's absolute position; the tokens before the first failure are kept.  Then the whole workgroup draws
// the next token: from the residual distribution norm(max(0, p - q)) of the failed position, or, when every token passed,
// from the target's row after the last one; both as argmax(log weight + Gumbel noise).
__global__ __launch_bounds__(1024) void accept_spd_kernel(TreeView tree, const float* __restrict__ logits, const float* __restrict__ lse,
                                                         const float* __restrict__ qrows, int V, const int32_t* __restrict__ len, int gamma,
                                                         uint64_t seed, AcceptView out) {
  __shared__ int eta_s;
  __shared__ uint64_t sh[16];
  const int s = blockIdx.x, M = tree.M;
  const int32_t* tok = tree.tok + (int64_t)s * M;
  if (threadIdx.x == 0) {
    int eta = gamma;
    for (int t = 1; t <= gamma; ++t) {
      int x = tok[t];
      if (x < 0 || x >= V) x = 0;
      const float lp = logits[((int64_t)s * M + t - 1) * V + x] - lse[s * M + t - 1];
      const float lq = qrows[((int64_t)s * gamma + t - 1) * V + x];
      const float u = uniform01(noise_key(seed, s * STREAMS_PER_SEQ + STREAM_ACCEPT, len[s] + t), 0);
      if (!(logf(u) < fminf(0.f, lp - lq))) { eta = t - 1; break; }
    }
    eta_s = eta;
    out.eta[s] = eta;
    out.bonus_row[s] = eta;
    out.out_cnt[s] = eta + 1;
    for (int i = 0; i < gamma; ++i) out.path[s * gamma + i] = i < eta ? i + 1 : -1;
    for (int i = 0; i < eta; ++i) out.out_tok[s * (gamma + 1) + i] = tok[i + 1];
  }
  __syncthreads();
  const int eta = eta_s;
  const float* prow = logits + ((int64_t)s * M + eta) * V;
  const float pl = lse[s * M + eta];
  const float* qrow = qrows + ((int64_t)s * gamma + (eta < gamma ? eta : 0)) * V;
  const uint64_t nk = noise_key(seed, s * STREAMS_PER_SEQ + STREAM_BONUS, len[s] + 1 + eta);
  float bk = -INFINITY;
  int bi = 0x7FFFFFFF;
  for (int v = threadIdx.x; v < V; v += (int)blockDim.x) {
    const float lp = prow[v] - pl;
    float k;
    if (eta < gamma) {
      const float w = expf(lp) - expf(qrow[v]);
      k = w > 0.f ? logf(w) : -INFINITY;
    } else {
      k = lp;
    }
    k += gumbel(nk, (uint64_t)v);
    if (better(k, v, bk, bi)) { bk = k; bi = v; }
  }
  bi = rank_idx(block_max_rank(rank_of(bk, bi), sh));
  if (bi < 0 || bi >= V) bi = 0;  // only reachable with non-finite rows: stay in the vocabulary
  if (threadIdx.x == 0) {
    out.bonus_tok[s] = bi;
    out.out_tok[s * (gamma + 1) + eta] = bi;
  }
}

hipError_t launch_accept_spd(TreeView tree, const float* logits, const float* lse, const float* qrows, int V, const int32_t* len, int B,
                             int gamma, uint64_t seed, AcceptView out, hipStream_t s) {
  hipLaunchKernelGGL(accept_spd_kernel, dim3(B), dim3(1024), 0, s, tree, logits, lse, qrows, V, len, gamma, seed, out);
  return hipGetLastError();
}

// ---- warped distributions -------------------------------------------------------------------------------------

// One workgroup per logits row: the row becomes the row of log p~ of the warped distribution (appendix
// "Hyper-parameter Details": the top_k most likely tokens, normalised; of those, in descending order, the shortest
// prefix whose cumulative probability exceeds top_p; normalised again), minus infinity outside the support, and the
// row's logsumexp becomes 0, so that every consumer of (logits, lse) rows works on p~ unchanged.  Entries rank by value
// descending, token id ascending; a NaN ranks last.
//   1. every wave's largest value; t = the top_k-th largest of those 16.  The top_k entries of the row reach t, and so do few
//      others (10 to 60 in a row of logits in no order): they are listed in LDS.
//   2. a row whose largest values share a few waves, or that repeats one value, lists more than WARP_SHORT or has no such t: a
//      threshold of value and id is then the top_k-th best of the threads' best entries, in top_k rounds of a workgroup-wide maximum, and
//      at most top_k * V / 1024 entries reach it
//   3. wave 0 orders the list (up to 64 entries: every lane counts the entries before its own) and does the arithmetic, one token per
//      lane, sums in descending order
// Bound by its chain of steps, one compute unit per row; 32000 tokens, top_k 10: 15.2 us with the threshold, the list and the order
// taken on 64-bit (value, id) ranks, 10.7 on values, ranks only in the list.  The first 32768 entries of the row live in registers.
// WARP_SHORT 128 / 512 / 2048, 4 rows with their copy, us (ranks): 1000 tokens in two waves, top_k 10 21.5 / 15.1 / 15.1; 4096 of one value,
// top_k 16 28.5 / 28.5 / 42.3; 8192 with the best 1024 in two waves 22.7 / 22.7 / 31.6; 151936 sorted 105 / 105 / 89.
constexpr int WARP_MAXK = 16, WARP_LIST = 2048, WARP_SHORT = 512;
__device__ __forceinline__ float lane_value(float v, int i) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), i)); }  // i uniform
__global__ __launch_bounds__(1024) void warp_rows_kernel(float* __restrict__ logits, float* __restrict__ lse, int V, int top_k, float top_p) {
  __shared__ uint64_t sh[2][16];
  __shared__ uint64_t list[WARP_LIST];
  __shared__ float best_s[16];
  __shared__ int count;
  __shared__ float tv[WARP_MAXK];
  __shared__ int ti[WARP_MAXK], keep_s;
  float* row = logits + (int64_t)blockIdx.x * V;
  const int t = threadIdx.x, lane = t & 63, k = min(min(top_k, WARP_MAXK), V);
  constexpr int PT = 32;
  float x[PT];
#pragma unroll
  for (int j = 0; j < PT; ++j) x[j] = row[min(t + 1024 * j, V - 1)];
  auto at = [&](int v) {  // entries beyond the registers
    const float y = row[v];
    return (y == y) ? y : -INFINITY;
  };
  if (t == 0) count = 0;
  float mine = -INFINITY;
#pragma unroll
  for (int j = 0; j < PT; ++j) {
    x[j] = (x[j] == x[j] && t + 1024 * j < V) ? x[j] : -INFINITY;
    mine = fmaxf(mine, x[j]);
  }
  for (int v = t + 1024 * PT; v < V; v += 1024) mine = fmaxf(mine, at(v));
  // a row that lies in registers whole is overwritten now, while the rest runs
  const bool held = V <= 1024 * PT;
  if (held)
    for (int v = t; v < V; v += 1024) row[v] = -INFINITY;
  const float wave_best = wave_max(mine);
  if (lane == 0) best_s[t >> 6] = wave_best;
  __syncthreads();
  float T;
  {
    const float w = best_s[lane & 15];
    int above = 0;
#pragma unroll
    for (int i = 0; i < 16; ++i) above += best_s[i] > w;
    T = -wave_max(above < k ? -w : -INFINITY);
  }
  const bool sparse = T > -INFINITY;  // uniform over the workgroup
  if (sparse && wave_best >= T) {     // uniform over the wave
#pragma unroll
    for (int j = 0; j < PT; ++j) {
      const uint64_t hits = __ballot(x[j] >= T);
      if (hits) {
        int at0 = 0;
        if (lane == 0) at0 = atomicAdd(&count, __popcll(hits));
        at0 = __builtin_amdgcn_readfirstlane(at0);
        if (at0 > WARP_SHORT) break;  // too long already
        const int o = at0 + __builtin_amdgcn_mbcnt_hi((uint32_t)(hits >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)hits, 0));
        if (x[j] >= T && o < WARP_LIST) list[o] = rank_of(x[j], t + 1024 * j);
      }
    }
    for (int v = t + 1024 * PT; v < V && *(volatile int*)&count <= WARP_SHORT; v += 1024) {
      const float y = at(v);
      if (y >= T) {
        const int o = atomicAdd(&count, 1);
        if (o < WARP_LIST) list[o] = rank_of(y, v);
      }
    }
  }
  __syncthreads();
  int n = count;
  if (n > WARP_SHORT || !sparse) {
    __syncthreads();
    if (t == 0) count = 0;
    uint64_t best = rank_of(-INFINITY, 0x7FFFFFFF);
#pragma unroll
    for (int j = 0; j < PT; ++j) {
      const uint64_t r = rank_of(x[j], t + 1024 * j);
      if (t + 1024 * j < V && r > best) best = r;
    }
    for (int v = t + 1024 * PT; v < V; v += 1024) {
      const uint64_t r = rank_of(at(v), v);
      if (r > best) best = r;
    }
    uint64_t R = 0, left = best;
    const int rounds = min(k, min(V, 1024));  // threads with an entry
    for (int r = 0; r < rounds; ++r) {
      R = block_max_rank(left, sh[r & 1]);  // (everybody has read the other buffer before this one's barrier)
      if (left == R) left = 0;
    }
    __syncthreads();
    if (best >= R) {
#pragma unroll
      for (int j = 0; j < PT; ++j) {
        const uint64_t r = rank_of(x[j], t + 1024 * j);
        if (t + 1024 * j < V && r >= R) {
          const int o = atomicAdd(&count, 1);
          if (o < WARP_LIST) list[o] = r;
        }
      }
      for (int v = t + 1024 * PT; v < V; v += 1024) {
        const uint64_t r = rank_of(at(v), v);
        if (r >= R) {
          const int o = atomicAdd(&count, 1);
          if (o < WARP_LIST) list[o] = r;
        }
      }
    }
    __syncthreads();
    n = count;
  }
  if (n > WARP_LIST) {  // only with more than 131072 tokens, and rows whose best entries share a few threads: one token a round
    uint64_t prev = ~0ull;
    for (int r = 0; r < k; ++r) {
      uint64_t b = 0;
      for (int v = t; v < V; v += 1024) {
        const uint64_t rk = rank_of(at(v), v);
        if (rk < prev && rk > b) b = rk;
      }
      prev = block_max_rank(b, sh[r & 1]);
      if (t == 0) list[r] = prev;
    }
    n = k;
    __syncthreads();
  }
  if (t < 64) {
    uint64_t own = 0;  // lane i keeps the i-th best
    if (n <= 64) {
      const uint64_t e = lane < n ? list[lane] : 0;
      const int lo = (int)(uint32_t)e, hi = (int)(e >> 32);
      int before = 0;
      for (int i = 0; i < n; ++i) {
        const uint64_t o = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane(hi, i) << 32) | (uint32_t)__builtin_amdgcn_readlane(lo, i);
        before += o > e;
      }
      if (lane < n && before < k) sh[0][before] = e;
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
      if (lane < k) own = ((volatile uint64_t*)sh[0])[lane];
    } else {
      auto lane_best = [&]() {
        uint64_t b = 0;
        for (int o = lane; o < n; o += 64) b = list[o] > b ? list[o] : b;
        return b;
      };
      uint64_t b = lane_best();
      for (int r = 0; r < k; ++r) {
        const uint64_t w = wave_max_rank(b);
        if (lane == r) own = w;
        if (b == w) {
          for (int o = lane; o < n; o += 64)
            if (list[o] == w) list[o] = 0;
          b = lane_best();
        }
      }
    }
    const bool in = lane < k;
    const float v = in ? rank_key(own) : -INFINITY, top = lane_value(v, 0);
    const float e = in ? expf(v - top) : 0.f;
    float S = 0.f;
    for (int i = 0; i < k; ++i) S += lane_value(e, i);
    const float p = e / S;
    float c = 0.f;
    int K = k;
    for (int i = 0; i < k; ++i) {
      c += lane_value(p, i);
      if (K == k && c > top_p) K = i + 1;
    }
    float s2 = 0.f;
    for (int i = 0; i < K; ++i) s2 += lane_value(p, i);
    if (in) {
      tv[lane] = logf(p / s2);
      ti[lane] = rank_idx(own);
    }
    if (lane == 0) {
      keep_s = K;
      lse[blockIdx.x] = 0.f;
    }
  }
  if (!held) {
    __syncthreads();  // wave 0 does not read the row, but others may still be listing it
    for (int v = t; v < V; v += 1024) row[v] = -INFINITY;
  }
  __syncthreads();
  // an entry's new value is written by the thread that overwrote its old one: one thread's stores to an address stay in order
  for (int i = 0; i < keep_s; ++i)
    if ((ti[i] & 1023) == t && ti[i] >= 0 && ti[i] < V) row[ti[i]] = tv[i];
}

hipError_t launch_warp_rows(float* logits, float* lse, int rows, int V, int top_k, float top_p, hipStream_t s) {
  if (rows <= 0) return hipSuccess;
  hipLaunchKernelGGL(warp_rows_kernel, dim3(rows), dim3(1024), 0, s, logits, lse, V, top_k, top_p);
  return hipGetLastError();
}

// ---- KV commit / rollback -------------------------------------------------------------------------------------

// grid (n_layers, B, 2): z = 0 keys, 1 values.  Every thread owns a fixed set of element offsets within a
// token's K (or V) and moves them for path depth 1, 2, ... in order; a destination slot is never the source
// of a later move, and earlier sources have been read already, so the in-place gather is race free.
template <typename T>
__global__ __launch_bounds__(256) void kv_gather_kernel(KvView kv, const int32_t* __restrict__ eta_p, const int32_t* __restrict__ path,
                                                        const int32_t* __restrict__ src_beam, const int32_t* __restrict__ cu_cnt,
                                                        int M, int gamma, int beam, int is_draft) {
  const int layer = blockIdx.x, s = blockIdx.y;
  T* base = (T*)(blockIdx.z ? kv.v : kv.k) + (int64_t)layer * kv.layer_stride;
  const int n = kv.len[s];
  const int eta = eta_p[s];
  const int row_elems = kv.n_kv_heads * kv.head_dim;
  const int cap = kv_capacity(kv);
  int cnt = 0, depth_max = eta;
  if (is_draft) {
    cnt = cu_cnt[s];
    if (cnt < 1 || cnt > gamma + 1) cnt = 1;
    depth_max = min(eta, gamma - 1);
  }
  for (int i = 1; i <= depth_max; ++i) {
    const int row = path[s * gamma + i - 1];
    if (row < 1 || row >= M) return;
    int src, dst;
    if (is_draft) {
      src = n + cnt + (i - 1) * beam + src_beam[s * M + row];
      dst = n + cnt - 1 + i;
    } else {
      src = n + row;
      dst = n + i;
    }
    if (src == dst) continue;
    if (src >= cap || dst >= cap) return;
    const T* sp = base + kv_token_offset(kv, s, src);
    T* dp = base + kv_token_offset(kv, s, dst);
    for (int e = threadIdx.x; e < row_elems; e += 256) dp[e] = sp[e];
  }
}

hipError_t launch_kv_gather(int dtype, KvView kv, int n_layers, int B, const int32_t* eta, const int32_t* path, const int32_t* src_beam,
                            const int32_t* cu_cnt, int M, int gamma, int beam, int is_draft, hipStream_t s) {
  dim3 grid(n_layers, B, 2);
  if (dtype == 1) hipLaunchKernelGGL((kv_gather_kernel<bf16_t>), grid, dim3(256), 0, s, kv, eta, path, src_beam, cu_cnt, M, gamma, beam, is_draft);
  else hipLaunchKernelGGL((kv_gather_kernel<float>), grid, dim3(256), 0, s, kv, eta, path, src_beam, cu_cnt, M, gamma, beam, is_draft);
  return hipGetLastError();
}

// Multi-token joint decoding (Section 3.1): the chain of the beam search is the output.  Written as an accept record
// whose last token plays the part of the bonus token: the first gamma - 1 tokens were run by the beam steps (their rows
// are gathered by the commit), the last one was not and becomes the pending token.
__global__ void accept_chain_kernel(TreeView tree, int B, int gamma, AcceptView out) {
  const int s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= B) return;
  const int32_t* tok = tree.tok + (int64_t)s * tree.M;
  out.eta[s] = gamma - 1;
  out.bonus_row[s] = gamma - 1;
  out.bonus_tok[s] = tok[gamma];
  out.out_cnt[s] = gamma;
  for (int i = 0; i < gamma; ++i) {
    out.path[s * gamma + i] = i < gamma - 1 ? i + 1 : -1;
    out.out_tok[s * (gamma + 1) + i] = tok[i + 1];
  }
}

hipError_t launch_accept_chain(TreeView tree, int B, int gamma, AcceptView out, hipStream_t s) {
  hipLaunchKernelGGL(accept_chain_kernel, dim3((B + 63) / 64), dim3(64), 0, s, tree, B, gamma, out);
  return hipGetLastError();
}

// lengths and the state of the next iteration
__global__ void commit_state_kernel(int32_t* tlen, int32_t* dlen, TreeView tree, AcceptView acc, int32_t* root_tok, int32_t* cu_tok,
                                    int32_t* cu_cnt, int B, int gamma, int tcap, int dcap) {
  const int s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= B) return;
  const int eta = acc.eta[s], t = acc.bonus_tok[s];
  if (tlen) tlen[s] = min(tcap, tlen[s] + eta + 1);
  if (dlen) {
    int cnt = cu_cnt[s];
    if (cnt < 1 || cnt > gamma + 1) cnt = 1;
    dlen[s] = min(dcap, dlen[s] + cnt + min(eta, gamma - 1));
  }
  root_tok[s] = t;
  if (eta == gamma) {
    const int row = acc.path[s * gamma + gamma - 1];
    cu_tok[s * (gamma + 1) + 0] = (row >= 0 && row < tree.M) ? tree.tok[(int64_t)s * tree.M + row] : 0;
    cu_tok[s * (gamma + 1) + 1] = t;
    cu_cnt[s] = 2;
  } else {
    cu_tok[s * (gamma + 1) + 0] = t;
    cu_cnt[s] = 1;
  }
}

hipError_t launch_commit_state(int32_t* tlen, int32_t* dlen, TreeView tree, AcceptView acc, int32_t* root_tok, int32_t* cu_tok,
                               int32_t* cu_cnt, int B, int gamma, int tcap, int dcap, hipStream_t s) {
  hipLaunchKernelGGL(commit_state_kernel, dim3((B + 63) / 64), dim3(64), 0, s, tlen, dlen, tree, acc, root_tok, cu_tok, cu_cnt, B, gamma,
                     tcap, dcap);
  return hipGetLastError();
}

}  // namespace mtad
