// The decoder pass of a small model over at most 8 rows in ONE launch: a draft's beam step, a chain or a single token of a model
// whose layers are a few megabytes.  Such a pass is bound by neither memory nor arithmetic: with a launch per step every step costs
// a launch, the ramp of its loads and the drain of its stores, about 4 us, for a fraction of a microsecond of work.
//
//   * Workgroups are persistent, one a compute unit, and own the same units (one or two strips of 16 features of a product, one (key
//     split, key head, sequence) of attention) in every layer.  A unit requests its weights, or its keys and values, before it
//     waits for what the step before it makes.
//   * A step hands its results on as words of 32 bits of payload and a 32-bit tag (relay.h), which everybody who needs them polls
//     past the caches until the tag is the one of this pass and layer: a hand-over is one store's way to memory and one load's way
//     back, with no acknowledgement, counter or flag between.  Measured, all to all, one addition: 1.3 us a step for 768 words
//     between 48 workgroups, 1.8 for 2048 words between 96, 2.9 for 8192; words of one line written by several workgroups take twice
//     as long, so a unit's results are whole lines.
//   * Every result of a step depends on all results of the step before, so nobody can be more than a step ahead of anybody's reads,
//     and two layers' words alternate.
//   * All units of a layer must run before the next can: the workgroups have to be on the machine at the same time.  Where another
//     launch holds the compute units that some of them need, whoever has waited too long in layer 0 counts those that have started.  If some
//     have not, the others share all units among themselves from the first layer on, with words of their own (nothing they write differs
//     from what was there); if all have, or one has been past layer 0 and so has seen a result of everybody, the pass goes on and nobody
//     counts again.  Every wait ends, at the latest after 0.2 s of this one wait with the status bit of a pass that was given up.
#include "attn_mfma_device.h"
#include "gemm.h"
#include "gemm_device.h"
#include "relay.h"

#include <atomic>
#include <utility>

namespace mtad {

namespace {

constexpr int RT = 512, RWAVES = RT / 64;
constexpr int TILES = 16;                      // bf16: weight tiles of a wave, all requested ahead: reductions of up to 4096 terms, with two strips 2048
constexpr int QUADS = 16;                      // float32: weight quads of a lane: up to 2048 terms, with two strips 1024
__host__ __device__ constexpr int most_terms(bool bf, int strips) { return (bf ? TILES * 32 : QUADS * 16) * RWAVES / strips; }
constexpr int PAIR_CHUNK = 8;                  // attention: most (query head, row) pairs of a unit (float32: half or a quarter of them)
constexpr int ROPE_SLOTS = 4;
constexpr int RELAY_BLOCKS = RWAVES;           // attention: blocks of keys of a split, one a wave; longer contexts get another one
constexpr int RELAY_MAX_LDS = 128 * 1024;      // a staged input, beside the static arrays
constexpr int RELAY_STRIPS = 128;              // products of more strips take two a unit: the fewer workgroups poll, the sooner words arrive

typedef const __attribute__((address_space(4))) RelayArgs* RelayPtr;
template <typename T>
__device__ __forceinline__ T ldc(const __attribute__((address_space(4))) T* p) {
  T v;
  __builtin_memcpy(&v, p, sizeof(T));
  return v;
}

__device__ __forceinline__ void put(uint64_t* p, uint32_t tag, float v) {
  __hip_atomic_store(p, ((uint64_t)tag << 32) | __float_as_uint(v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t get(const uint64_t* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ uint32_t get32(const uint32_t* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ bool tagged(uint64_t w, uint32_t tag) { return (uint32_t)(w >> 32) == tag; }
__device__ __forceinline__ float payload(uint64_t w) { return __uint_as_float((uint32_t)w); }

struct RelaySmem {
  float red[2][RWAVES][RELAY_MAX_ROWS][16];  // products: a wave's share, [strip][wave][row][feature]
  float ssq[2][RWAVES];                      // sums of squares of a wave's share of a row, two units in turn
  float2 rope[ROPE_SLOTS][2 * RELAY_MAX_ROWS * 8];  // [strip][row][pair] of a unit
  int rope_unit[ROPE_SLOTS];
  float m[RWAVES][PAIR_CHUNK], l[RWAVES][PAIR_CHUNK], own[RELAY_MAX_ROWS][PAIR_CHUNK];  // attention: of a wave's keys; scores of the own rows
  int leave;
  uint32_t verdict;
};

// What a wait has to know besides its words
struct Watch {
  uint32_t *sync, *status;
  uint32_t epoch;
  unsigned patience, give_up;
  int groups, group;
  bool again;      // one of those that started over
  bool committed;  // this workgroup has had input of a layer above 0: every workgroup has done its share of layer 0
  bool settled;    // they have been counted, and the pass goes on: nobody counts again
};
__device__ __forceinline__ uint64_t* rank_word(uint32_t* sync, int b) { return (uint64_t*)(sync + 64 + RELAY_MAX_GROUPS) + b; }

// What a rank word says of this pass: that it goes on (no workgroups), or who starts over
__device__ __forceinline__ bool goes_on(uint32_t word) { return word >> 16 == 0; }

// Counts the workgroups that are there, and says in all rank words what becomes of the pass.  One wave of whoever has waited too long; the
// first in a pass does it.  A workgroup that is counted (state 3) finds out when it commits or ends, and looks at its rank word then.
__device__ __forceinline__ void count_in(const Watch& c, int lane) {
  int mine = 0;
  if (lane == 0) mine = __hip_atomic_exchange(c.sync + 2, c.epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != c.epoch;
  if (!__builtin_amdgcn_readfirstlane(mine)) return;
  int n = 0, done = 0;
  bool past = false;  // somebody has been past layer 0
  unsigned in = 0;    // bit i: workgroup i * 64 + lane
  for (int i = 0; i < RELAY_MAX_GROUPS / 64; ++i) {
    uint32_t was = c.epoch * 4 + 1;
    const int b = i * 64 + lane;
    const bool got = b < c.groups && __hip_atomic_compare_exchange_strong(c.sync + 64 + b, &was, c.epoch * 4 + 3, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    in |= (unsigned)got << i;
    n += __popcll(__ballot(got));
    done += __popcll(__ballot(b < c.groups && !got && was == c.epoch * 4));
    past = past || __any(b < c.groups && !got && was == c.epoch * 4 + 2);
  }
  const bool on = past || n + done == c.groups;
  if (!on && lane == 0) __hip_atomic_fetch_add(c.sync + 3, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  int before = 0;
  for (int i = 0; i < RELAY_MAX_GROUPS / 64; ++i) {
    const int b = i * 64 + lane;
    const bool got = (in >> i) & 1;
    const unsigned long long all = __ballot(got);
    const int rank = got ? before + __popcll(all & ((1ull << lane) - 1)) : 0xFFFF;
    if (b < c.groups) __hip_atomic_store(rank_word(c.sync, b), (uint64_t)c.epoch << 32 | (on ? 0u : (uint32_t)n << 16 | (uint32_t)rank), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    before += __popcll(all);
  }
}

// Now and then during a wait (all lanes of a wave): is it over for another reason than its words?  since: when this was first asked in it, 0 before.
__device__ __forceinline__ bool must_leave(const Watch& c, int lane, unsigned long long& since) {
  if (get32(c.sync + 1) == c.epoch) return true;
  if (!c.again) {
    const uint64_t word = get(rank_word(c.sync, c.group));
    if ((uint32_t)(word >> 32) == c.epoch && !goes_on((uint32_t)word)) return true;
  }
  const unsigned long long now = wall_clock64();
  if (!since) since = now;
  const unsigned long long waited = now - since;
  if (waited > c.give_up) {
    if (lane == 0) {
      atomicOr(c.status, (uint32_t)ST_TIMEOUT);
      __hip_atomic_store(c.sync + 1, c.epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    return true;
  }
  return !c.again && !c.committed && !c.settled && waited > c.patience;
}

// This workgroup has had input of layer l: above 0, it says so, once.  was: what its state was (thread 0; needed at the end only).
__device__ __forceinline__ void commit(Watch& c, int l, int tid, int& was) {
  if (l == 0 || c.again || c.committed) return;
  c.committed = true;
  if (tid == 0) was = (int)__hip_atomic_exchange(c.sync + 64 + c.group, c.epoch * 4 + 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Brings this lane's words at(i) with that tag; also: what else is requested in every turn.  False: leave.  (How many words is a
// constant: a branch around every one of eight costs more than the words.)
struct Nothing {
  __device__ __forceinline__ void operator()() const {}
};
template <int N, typename At, typename Also = Nothing>
__device__ __forceinline__ bool collect(uint64_t (&w)[N], At at, uint32_t tag, const Watch& c, int lane, Also also = Also()) {
  unsigned long long since = 0;
#pragma unroll 1
  for (int turns = 1;; ++turns) {
    also();
#pragma unroll
    for (int i = 0; i < N; ++i) w[i] = get(at(i));
    uint32_t differ = 0;
#pragma unroll
    for (int i = 0; i < N; ++i) differ |= (uint32_t)(w[i] >> 32) ^ tag;
    const bool there = differ == 0;
    if (__all(there)) return true;
    if ((turns & 31) == 0 && must_leave(c, lane, since)) return false;
  }
}

// ---- products ------------------------------------------------------------------------------------------------------

template <bool BF>
struct Weights;
template <>
struct Weights<true> {
  Frag w[TILES];
};
template <>
struct Weights<false> {
  float4 w[QUADS];
};

struct Unit {  // a product unit: strips nt .. nt + ns - 1
  const void* W;
  int nt, ns, N, K;
};

// float32 models: row of the weight matrix that is feature j (0 .. 15) of strip nt
__device__ __forceinline__ int f32_row(int step, int nt, int j, int N, int hd) {
  if (step == RS_QKV) {
    const int tph = hd >> 4;
    return nt / tph * hd + (nt % tph) * 8 + (j & 7) + (j >> 3) * (hd >> 1);
  }
  if (step == RS_GU) return nt * 8 + (j & 7) + (j >> 3) * (N >> 1);
  return nt * 16 + j;
}

// This wave's part of the unit's weights, all of it.  bf16: every RWAVES-th k tile; float32: lane (quad of four, feature) of every
// RWAVES-th step of 16 terms.
template <bool BF>
__device__ __forceinline__ void request_weights(Weights<BF>& r, const Unit& u, int step, int wave, int hd, int lane) {
  auto strips = [&](auto NS_) {
    constexpr int NS = decltype(NS_)::value, T = (BF ? TILES : QUADS) / NS;
    if constexpr (BF) {
      const int KT = u.K >> 5;
      const char* const p = (const char*)u.W + ((size_t)u.nt * KT << 10);
#pragma unroll
      for (int i = 0; i < T; ++i)
        if (wave + i * RWAVES < KT) {
#pragma unroll
          for (int s = 0; s < NS; ++s) r.w[s * T + i].n = *(const uintx4*)(p + ((size_t)(s * KT + wave + i * RWAVES) << 10) + (unsigned)lane * 16u);
        } else if (wave + (i & ~3) * RWAVES < KT) {  // the rest of a group of four
#pragma unroll
          for (int s = 0; s < NS; ++s) r.w[s * T + i].n = uintx4{0, 0, 0, 0};
        }
    } else {
      const float* p[NS];
#pragma unroll
      for (int s = 0; s < NS; ++s) p[s] = (const float*)u.W + (int64_t)f32_row(step, u.nt + s, lane & 15, u.N, hd) * u.K + (lane >> 4) * 4;
#pragma unroll
      for (int i = 0; i < T; ++i) {
        const int k = (wave + i * RWAVES) * 16;
        if (k < u.K) {
#pragma unroll
          for (int s = 0; s < NS; ++s) {
            r.w[s * T + i] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (k + (lane >> 4) * 4 < u.K) r.w[s * T + i] = *(const float4*)(p[s] + k);
          }
        }
      }
    }
  };
  if (u.ns == 1) strips(std::integral_constant<int, 1>{});
  else strips(std::integral_constant<int, 2>{});
}

// The product of the unit's strips with the input in LDS; the waves' shares of it go to sm.red.
template <bool BF>
__device__ __forceinline__ void multiply(RelaySmem& sm, const unsigned char* x, Weights<BF>& r, const Unit& u, int step, int R, int hd, int wave, int lane) {
  const int c = lane & 15, kg = lane >> 4;
  auto strips = [&](auto NS_) {
    constexpr int NS = decltype(NS_)::value, T = (BF ? TILES : QUADS) / NS;
    if constexpr (BF) {
      const int KT = u.K >> 5;
      floatx4 acc[NS];
#pragma unroll
      for (int s = 0; s < NS; ++s) acc[s] = floatx4{0.f, 0.f, 0.f, 0.f};
      const unsigned char* const xl = x + ((kg * 2 + (c >> 3)) * R + min(c & 7, R - 1)) * 16;
#pragma unroll
      for (int i0 = 0; i0 < T; i0 += 4) {  // four tiles at a time; those past the end have no weights
        if (wave + i0 * RWAVES >= KT) break;
        {
          Frag b[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) b[i].n = *(const uintx4*)(xl + (unsigned)(min(wave + (i0 + i) * RWAVES, KT - 1) * (128 * R)));
#pragma unroll
          for (int i = 0; i < 4; ++i) {
#pragma unroll
              for (int s = 0; s < NS; ++s) acc[s] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(r.w[s * T + i0 + i].v, b[i].v, acc[s], 0, 0, 0);
            }
        }
      }
#pragma unroll
      for (int s = 0; s < NS; ++s) {  // columns c and c + 8 are the hi and lo terms of a row
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[s][e] += row_turn<8>(acc[s][e]);
        if (c < 8) *(floatx4*)&sm.red[s][wave][c][kg * 4] = acc[s];
      }
    } else {
      auto rows = [&](auto RB_) {
        constexpr int RB = decltype(RB_)::value;
        constexpr int NA = NS * RB <= 8 ? 4 : 2;  // sums of a lane: with one the pass's error is a tenth more than the steps'
        float acc[NS][RB][NA];
#pragma unroll
        for (int s = 0; s < NS; ++s)
#pragma unroll
          for (int m = 0; m < RB; ++m)
#pragma unroll
            for (int n = 0; n < NA; ++n) acc[s][m][n] = 0.f;
#pragma unroll
        for (int i = 0; i < T; ++i) {
          const int k = (wave + i * RWAVES) * 16;
          if (k >= u.K) break;
          {
            float4 v[RB];
#pragma unroll
            for (int m = 0; m < RB; ++m) v[m] = *(const float4*)((const float*)x + min(m, R - 1) * u.K + min(k + kg * 4, u.K - 4));
#pragma unroll
            for (int s = 0; s < NS; ++s) {
              const float4 w = r.w[s * T + i];
#pragma unroll
              for (int m = 0; m < RB; ++m) {
                float* const a = acc[s][m];
                a[0] = fmaf(w.x, v[m].x, a[0]);
                a[1] = fmaf(w.y, v[m].y, a[1]);
                a[NA - 2] = fmaf(w.z, v[m].z, a[NA - 2]);
                a[NA - 1] = fmaf(w.w, v[m].w, a[NA - 1]);
              }
            }
          }
        }
#pragma unroll
        for (int s = 0; s < NS; ++s)
#pragma unroll
          for (int m = 0; m < RB; ++m) {
            const float y = xsum<32>(xsum<16>(NA == 4 ? (acc[s][m][0] + acc[s][m][1]) + (acc[s][m][NA - 2] + acc[s][m][NA - 1]) : acc[s][m][0] + acc[s][m][1]));
            if (kg == 0) sm.red[s][wave][m][c] = y;
          }
      };
      if (R == 1) rows(std::integral_constant<int, 1>{});
      else if (R == 2) rows(std::integral_constant<int, 2>{});
      else if (R <= 4) rows(std::integral_constant<int, 4>{});
      else if (R <= 6) rows(std::integral_constant<int, 6>{});
      else rows(std::integral_constant<int, 8>{});
    }
  };
  if (u.ns == 1) strips(std::integral_constant<int, 1>{});
  else strips(std::integral_constant<int, 2>{});
}
__device__ __forceinline__ float result(const RelaySmem& sm, int s, int m, int j) {
  float v[RWAVES];
#pragma unroll
  for (int w = 0; w < RWAVES; ++w) v[w] = sm.red[s][w][m][j];
#pragma unroll
  for (int n = RWAVES / 2; n; n /= 2)  // (in pairs: a shorter chain, and less rounding)
#pragma unroll
    for (int w = 0; w < n; ++w) v[w] += v[w + n];
  return v[0];
}

// ---- attention -----------------------------------------------------------------------------------------------------

template <int HD>
struct AttnF32 {
  static constexpr int EPL = 4;                // dims per 16 bytes
  static constexpr int E = HD / 64;            // of those per lane, 64 dims apart
  static constexpr int KPL = 4;                // keys of a load, 16 lanes each
  static constexpr int NL = HD == 64 ? 16 : 8;  // loads of a block (K and V of one in registers)
  static constexpr int BK = NL * KPL;          // keys of a block
  static constexpr int PC = HD == 64 ? 4 : 2;  // most (query head, row) pairs of a unit
};

template <int J>
__device__ __forceinline__ int of_lane(int v) {  // the value of lane J of the 16 lanes of a key
  return __builtin_amdgcn_update_dpp(0, v, 0x150 + J, 0xf, 0xf, true);
}
// of 2N partial sums a lane keeps the N whose number has the lane's bit N and adds the partner's, N lanes away
template <int N>
__device__ __forceinline__ void halve_sums(float* y, int c) {
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
template <typename F, int... J>
__device__ __forceinline__ void each_of(F f, std::integer_sequence<int, J...>) {
  (f(std::integral_constant<int, J>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void each(F f) {
  each_of(f, std::make_integer_sequence<int, N>{});
}

// A query in this lane's dims
template <int N>
struct Query {
  float v[N];
  __device__ __forceinline__ void set(const float* p, int e) {  // dims 4 e .. + 3 of the lane's
    const float4 t = *(const float4*)p;
    v[4 * e] = t.x; v[4 * e + 1] = t.y; v[4 * e + 2] = t.z; v[4 * e + 3] = t.w;
  }
  __device__ __forceinline__ float dot(const uint4& k, int e, float sum) const {
    sum = fmaf(v[4 * e], __uint_as_float(k.x), sum);
    sum = fmaf(v[4 * e + 1], __uint_as_float(k.y), sum);
    sum = fmaf(v[4 * e + 2], __uint_as_float(k.z), sum);
    return fmaf(v[4 * e + 3], __uint_as_float(k.w), sum);
  }
};
__device__ __forceinline__ float element(const uint4& u, int i) { return __uint_as_float(i == 0 ? u.x : i == 1 ? u.y : i == 2 ? u.z : u.w); }

// (cos, sin) of an angle, accurate far beyond float32: the angle less a multiple of pi / 2, then the power series of both
__device__ __forceinline__ float2 turn_of(double ang) {
  const double k = rint(ang * 0.63661977236758134308);  // 2 / pi
  const double r = fma(k, -6.123233995736766036e-17, fma(k, -1.5707963267948965580, ang)), z = r * r;  // pi / 2 = the second + the first
  double s = 1.0 / 6227020800.0, c = 1.0 / 479001600.0;  // 13!, 12!
  s = fma(s, z, -1.0 / 39916800.0);
  s = fma(s, z, 1.0 / 362880.0);
  s = fma(s, z, -1.0 / 5040.0);
  s = fma(s, z, 1.0 / 120.0);
  s = fma(s, z, -1.0 / 6.0);
  s = fma(s * z, r, r);
  c = fma(c, z, -1.0 / 3628800.0);
  c = fma(c, z, 1.0 / 40320.0);
  c = fma(c, z, -1.0 / 720.0);
  c = fma(c, z, 1.0 / 24.0);
  c = fma(c, z, -0.5);
  c = fma(c, z, 1.0);
  const int quarter = (int)(long long)k & 3;
  const double cs = quarter & 1 ? s : c, sn = quarter & 1 ? c : s;
  return make_float2((float)(quarter == 1 || quarter == 2 ? -cs : cs), (float)(quarter >= 2 ? -sn : sn));
}

// ---- the pass ------------------------------------------------------------------------------------------------------

struct Step {  // where a layer's words are
  int l, groups;
  uint32_t tag;
  uint64_t *words;          // this layer's
  const uint64_t* h_words;  // the residual stream that the layer before left
};

// Keeps a value computed here, before a wait: left to itself the compiler moves such arithmetic to its use, behind the wait, where
// every instruction counts (a wave alone on its SIMD issues one in 4 to 8 clocks).  Offsets, not pointers: what comes out of here is
// no longer known to point to global memory or LDS.
template <typename T>
__device__ __forceinline__ void pin(T& v) {
  asm volatile("" : "+v"(v));
}

// One unit of a product.  fresh: its input is not in LDS yet.
template <bool BF, int HD>
__device__ __forceinline__ bool relay_product(RelaySmem& sm, unsigned char* x, RelayPtr A, Watch& watch, const Step& at, int step, int unit, bool fresh, int& parity, int& commit_was) {
  // What a unit derives from the thread index and the arguments is computed inside the unit, not kept in registers across all kinds
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  asm volatile("" : "+s"(A));
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int d = A->d, f = A->f, H = A->H, KVH = A->KVH, R = A->rows, l = at.l;
  const int wl = 1 + 6 * l;
  const bool normed = step == RS_QKV || step == RS_GU, embed = step == RS_QKV && l == 0, resid = !normed;
  Unit u;
  u.N = step == RS_QKV ? (H + 2 * KVH) * HD : step == RS_GU ? 2 * f : d;
  u.K = step == RS_O ? H * HD : step == RS_DOWN ? f : d;
  u.nt = unit * A->strips[step];
  u.ns = min(A->strips[step], (u.N >> 4) - u.nt);
  u.W = A->w[wl + (step == RS_QKV ? 1 : step == RS_O ? 2 : step == RS_GU ? 4 : 5)];
  Weights<BF> wts;
  request_weights<BF>(wts, u, step, wave, HD, lane);

  // ---- what the end of the unit needs, ahead of the wait: thread (strip s, row m, feature or pair j)
  const int per = resid ? 4 : 3, j = tid & ((1 << per) - 1), sr = tid >> per, s = sr / R, nt = u.nt + s;
  int m = sr - s * R;
  bool ends = s < u.ns;
  const int n = nt * 16 + j;
  unsigned out = 0;  // word where the result goes
  bool adds = false;
  unsigned before_at = 0;  // word that a residual step adds to
  const uint64_t* const before_words = step == RS_O ? at.h_words : at.words + A->mail.hm;
  const uint32_t before_tag = step == RS_O ? at.tag - 1 : at.tag;
  uint64_t before = 0;
  float2 cs = make_float2(1.f, 0.f);
  bool turned = false;  // q and k heads are rotated
  typedef typename std::conditional<BF, kv16_t, float>::type T;  // of the cache
  int64_t cache = -1;  // element of the cache
  bool is_kv = false, is_k = false;
  const float eps = A->eps;
  const bool last = l + 1 == A->n_layers;
  if (resid) {
    out = (unsigned)((step == RS_O ? A->mail.hm : A->mail.hd) + m * d + n);
    if (step == RS_O && l == 0) {
      if (ends) {
        int64_t token = A->rd.tok[m];
        if (token < 0 || token >= A->vocab) token = 0;  // inactive rows carry no meaningful token
        if constexpr (BF) before = (uint64_t)((const bf16_t*)A->w[0])[token * d + n] << 16;
        else before = __float_as_uint(((const float*)A->w[0])[token * d + n]);
      }
    } else {
      adds = ends;
      before_at = (unsigned)(m * d + n);
    }
  } else if (step == RS_GU) {
    out = (unsigned)(A->mail.act + m * f + nt * 8 + j);
  } else {
    out = (unsigned)(A->mail.qkv + m * u.N + nt * 16 + j);
    constexpr int TPH = HD >> 4;
    const int head = nt / TPH, i = (nt % TPH) * 8 + j;
    // the rotary table of the unit's rows and pairs, kept from layer to layer
    const int slot_r = (unit / at.groups) % ROPE_SLOTS;
    if (sm.rope_unit[slot_r] != unit) {  // (the same in all threads: read before and written after a barrier)
      __syncthreads();
      if (ends) sm.rope[slot_r][tid] = turn_of((double)A->rd.pos[m] * A->inv_freq[i]);
      if (tid == 0) sm.rope_unit[slot_r] = unit;
    }
    turned = head < H + KVH;
    if (ends && turned) cs = sm.rope[slot_r][tid];  // (written by this thread)
    is_kv = head >= H;
    if (ends && is_kv) {
      const int slot = A->rd.slot[m];
      const KvView kv = ldc(&A->kv);
      if (slot >= kv_capacity(kv)) {
        atomicOr(watch.status, (uint32_t)ST_KV_CAP);
      } else if (slot >= 0) {
        is_k = head < H + KVH;
        cache = (int64_t)l * kv.layer_stride + kv_token_offset(kv, m / A->Rseq, slot) + (int64_t)(head - (is_k ? H : H + KVH)) * HD + i;
      }
    }
  }
  const int wpr = R == 1 ? 8 : R == 2 ? 4 : R <= 4 ? 2 : 1;  // waves of a row while the input is brought
  pin(m);
  pin(out);
  pin(before_at);
  pin(cache);
  pin(cs.x);
  pin(cs.y);

  // ---- the input
  if (fresh) {
    const uint64_t* const src = step == RS_QKV ? at.h_words : at.words + (step == RS_O ? A->mail.att : step == RS_GU ? A->mail.hm : A->mail.act);
    const uint32_t src_tag = step == RS_QKV ? at.tag - 1 : at.tag;
    const float* const gain = (const float*)A->w[wl + (step == RS_GU ? 3 : 0)];
    const int my_row = wave / wpr, my_part = wave % wpr;
    parity ^= 1;
    bool stay = true;
    float ss = 0.f;
    if (my_row < R) {
      const int stride = wpr * 64, half_k = u.K >> 1;
      int64_t token = 0;
      if (embed) {
        token = A->rd.tok[my_row];
        if (token < 0 || token >= A->vocab) token = 0;
      }
      // lane: pairs first + i stride of a batch; those past the end are the last one again, and not staged
      auto bring = [&](auto N_) {
        constexpr int N = decltype(N_)::value;
#pragma unroll 1
        for (int j0 = my_part * 64; j0 < half_k && stay; j0 += stride * N) {
          const int first = j0 + lane;
          unsigned at_x = BF ? (unsigned)((((first >> 2) * 2 * R + my_row) * 8 + (first & 3) * 2) * 2) : (unsigned)((my_row * u.K + 2 * first) * 4);
          const unsigned step_x = BF ? (unsigned)(stride * R * 8) : (unsigned)(stride * 8);
          unsigned at_w[N];
#pragma unroll
          for (int i = 0; i < N; ++i) at_w[i] = (unsigned)min(first + i * stride, half_k - 1) * 16;
          pin(at_x);
          uint64_t w[2 * N];
          float2 g[N];
          if (normed) {
#pragma unroll
            for (int i = 0; i < N; ++i) g[i] = *(const float2*)((const char*)gain + (at_w[i] >> 1));
          }
          if (embed) {
#pragma unroll
            for (int i = 0; i < N; ++i) {
              if constexpr (BF) {
                const uint32_t two = *(const uint32_t*)((const char*)((const bf16_t*)A->w[0] + token * d) + (at_w[i] >> 2));
                w[2 * i] = two << 16;
                w[2 * i + 1] = two & 0xFFFF0000u;
              } else {
                const uint2 two = *(const uint2*)((const char*)((const float*)A->w[0] + token * d) + (at_w[i] >> 1));
                w[2 * i] = two.x;
                w[2 * i + 1] = two.y;
              }
            }
          } else {
            const char* const p = (const char*)(src + (size_t)my_row * u.K);
            stay = collect(w, [&](int i) { return (const uint64_t*)(p + at_w[i >> 1] + (i & 1) * 8); }, src_tag, watch, lane,
                           [&]() { if (adds) before = get(before_words + before_at); });  // (what is added to came long before)
          }
#pragma unroll
          for (int i = 0; i < N; ++i)
            if (first + i * stride < half_k) {
              float a = payload(w[2 * i]), b = payload(w[2 * i + 1]);
              if (normed) {
                ss = fmaf(a, a, ss);
                ss = fmaf(b, b, ss);
                a *= g[i].x;
                b *= g[i].y;
              }
              unsigned char* const to = x + at_x + i * step_x;
              if constexpr (BF) {
                typedef float f2 __attribute__((ext_vector_type(2)));
                typedef __bf16 b2 __attribute__((ext_vector_type(2)));
                const f2 v = {a, b};
                const b2 hi = __builtin_convertvector(v, b2);
                *(b2*)to = hi;
                *(b2*)(to + R * 16) = __builtin_convertvector(v - __builtin_convertvector(hi, f2), b2);
              } else {
                *(float2*)to = make_float2(a, b);
              }
            }
        }
      };
      const int n = (half_k - my_part * 64 + stride - 1) / stride;  // (stride: a power of two)
      if (n <= 1) bring(std::integral_constant<int, 1>{});
      else if (n == 2) bring(std::integral_constant<int, 2>{});
      else if (n == 3) bring(std::integral_constant<int, 3>{});
      else if (n <= 6 && n != 4) bring(std::integral_constant<int, 6>{});
      else bring(std::integral_constant<int, 8>{});
    }
    if (!stay) sm.leave = 1;
    if (normed) {
      ss = wave_sum(ss);
      if (lane == 0) sm.ssq[parity][wave] = ss;
    }
  }
  __syncthreads();
  const int leave = sm.leave;  // (seen to after the product)
  float inv = 1.0f;
  if (normed) {
    float ssq = 0.f;
#pragma unroll
    for (int w = 0; w < RWAVES; ++w) {
      const float t = sm.ssq[parity][w];
      ssq += (unsigned)(w - m * wpr) < (unsigned)wpr ? t : 0.f;
    }
    inv = 1.0f / sqrtf(ssq / (float)u.K + eps);
  }
  pin(inv);
  multiply<BF>(sm, x, wts, u, step, R, HD, wave, lane);
  if (!leave) commit(watch, l, tid, commit_was);
  __syncthreads();
  if (leave) return false;
  if (resid) {
    bool stay = true;
    unsigned long long since = 0;
    float hn = ends ? result(sm, s, m, j) : 0.f;
    for (int turns = 1; stay && __any(adds && !tagged(before, before_tag)); ++turns) {  // (there, but this load was the earlier one)
      if (adds && !tagged(before, before_tag)) before = get(before_words + before_at);
      if ((turns & 31) == 0 && must_leave(watch, lane, since)) stay = false;
    }
    if (!stay) sm.leave = 1;  // (seen by all after the next barrier)
    if (ends) hn += payload(before);
    if (step == RS_O || !last) {
      if (ends && stay) put(at.words + out, at.tag, hn);
    } else if constexpr (BF) {  // the lm_head's input, for the launch after this one
      float q = hn * hn;
      q += row_turn<8>(q);
      q += row_turn<4>(q);
      q += row_turn<2>(q);
      q += row_turn<1>(q);
      if (ends) {
        bf16_t hi, lo;
        split_bf16(hn * ((const float*)A->w[wl + 6])[n], hi, lo);
        A->xg[act_offset(A->ncg, R, d, 0, m, n)] = hi;
        A->xg[act_offset(A->ncg, R, d, 1, m, n)] = lo;
        if (j == 0) A->ssq[(int64_t)m * (d >> 4) + nt] = q;
      }
    } else {
      if (ends) A->h[(int64_t)m * d + n] = hn;
    }
    return true;
  }
  if (!ends) return true;
  const float y0 = result(sm, s, m, j), yp = result(sm, s, m, j + 8);
  float y1 = y0 * inv, y2 = yp * inv;
  if (step == RS_GU) {
    put(at.words + out, at.tag, y1 / (1.0f + expf(-y1)) * y2);
    return true;
  }
  if (turned) {
    const float t = fmaf(y1, cs.x, -(y2 * cs.y));
    y2 = fmaf(y2, cs.x, y1 * cs.y);
    y1 = t;
  }
  if (is_kv) {
    const T t1 = (T)y1, t2 = (T)y2;
    y1 = (float)t1;
    y2 = (float)t2;
    if (cache >= 0) {
      T* const to = (T*)(is_k ? A->kv.k : A->kv.v) + cache;
      to[0] = t1;
      to[HD >> 1] = t2;
    }
  }
  put(at.words + out, at.tag, y1);
  put(at.words + out + 8, at.tag, y2);
  return true;
}

// The waves' results [wave][pair][dim] and the own rows, added in order, and handed on; splits other than the first hand on theirs to the first.
template <bool BF, int HD, int PC>
__device__ __forceinline__ void relay_merge(RelaySmem& sm, const float* o_s, int o_stride, const float* vn, RelayPtr A, const Watch& watch, const Step& at, int split, int eff, int used,
                                            int seq, int kvh, int p0, int np, int wave, int lane) {
  auto exponential = [](float v) { return BF ? __builtin_amdgcn_exp2f(v) : expf(v); };
  const int H = A->H, KVH = A->KVH, Rseq = A->Rseq, G = H / KVH, P = G * Rseq, splits = A->splits;
  bool stay = true;
#pragma unroll 1
  for (int i0 = wave * 64; i0 < np * HD && stay; i0 += RT) {
    const int r = i0 / HD, p = p0 + r, dim = i0 % HD + lane;  // (64 divides HD: a wave's are of one pair)
    // lane w of a row of 16: wave w's, or own row w - 8's, maximum and sum; its share of the row's scale
    const int w16 = lane & 15;
    float m16 = -INFINITY, l16 = 1.f;
    if (w16 < used) {
      m16 = sm.m[w16][r];
      l16 = sm.l[w16][r];
    }
    if (w16 >= RWAVES && split == 0) m16 = sm.own[w16 - RWAVES][r];
    float M = fmaxf(m16, row_turn<8>(m16));
    M = fmaxf(M, row_turn<4>(M));
    M = fmaxf(M, row_turn<2>(M));
    M = fmaxf(M, row_turn<1>(M));
    const float e16 = m16 == -INFINITY ? 0.f : exponential(m16 - M);
    float sum = l16 * e16;
    sum += row_turn<8>(sum);
    sum += row_turn<4>(sum);
    sum += row_turn<2>(sum);
    sum += row_turn<1>(sum);
    float o = 0.f;
    if (used > 0) {
      float ow[RWAVES];
#pragma unroll
      for (int w = 0; w < RWAVES; ++w) ow[w] = o_s[min(w, used - 1) * o_stride + r * HD + dim];
#pragma unroll
      for (int w = 0; w < RWAVES; ++w) o = fmaf(ow[w], __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(e16), w)), o);
    }
    if (split == 0) {
      auto own = [&](auto N_) {
        constexpr int N = decltype(N_)::value;
        float vw[N];
#pragma unroll
        for (int w = 0; w < N; ++w) vw[w] = vn[min(w, Rseq - 1) * HD + dim];
#pragma unroll
        for (int w = 0; w < N; ++w) o = fmaf(vw[w], __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(e16), RWAVES + w)), o);
      };
      if (Rseq == 1) own(std::integral_constant<int, 1>{});
      else own(std::integral_constant<int, RELAY_MAX_ROWS>{});
    }
    uint64_t* const part = at.words + A->mail.part + (size_t)(((seq * KVH + kvh) * P + p) * splits) * (HD + 2);  // (max, sum, output) of every split
    if (split > 0) {
      uint64_t* const to = part + (size_t)split * (HD + 2);
      put(to + 2 + dim, at.tag, o);
      if (dim == 0) {
        put(to, at.tag, M);
        put(to + 1, at.tag, sum);
      }
      continue;
    }
    auto gather = [&](auto N_) {  // all splits' words at once
      constexpr int N = decltype(N_)::value;
      uint64_t w[3 * N];
      stay = collect(w, [&](int i) { return part + (size_t)min(1 + i / 3, eff - 1) * (HD + 2) + (i % 3 < 2 ? i % 3 : 2 + dim); }, at.tag, watch, lane);
      if (!stay) return;
#pragma unroll
      for (int s2 = 0; s2 < N; ++s2) {
        const float M2 = s2 + 1 < eff ? payload(w[3 * s2]) : -INFINITY;
        if (M2 == -INFINITY) continue;
        const float Mn = fmaxf(M, M2), wa = M == -INFINITY ? 0.f : exponential(M - Mn), wb = exponential(M2 - Mn);
        sum = sum * wa + payload(w[3 * s2 + 1]) * wb;
        o = o * wa + payload(w[3 * s2 + 2]) * wb;
        M = Mn;
      }
    };
    if (eff > 4) gather(std::integral_constant<int, RELAY_MAX_SPLITS - 1>{});
    else if (eff > 2) gather(std::integral_constant<int, 3>{});
    else if (eff > 1) gather(std::integral_constant<int, 1>{});
    if (stay) put(at.words + A->mail.att + (size_t)(seq * Rseq + p % Rseq) * (H * HD) + (kvh * G + p / Rseq) * HD + dim, at.tag, sum > 0.f ? o / sum : 0.f);
  }
  // Read between the next unit's barriers, or at the end of the run: a wave that read it here could do so after a faster one has failed the
  // next unit's wait, and the two would be at different barriers from then on.
  if (!stay) sm.leave = 1;
  __syncthreads();  // what was staged is free again
}

// One unit of attention: (split, group of pairs, key head, sequence), at most PC (query head, row) pairs; the split that merges is the last
// of its item's, as a workgroup with several of them would wait for itself otherwise.  The waves take blocks of
// cached keys in turn; the pass's own rows are keys in LDS.
//
// float32 models: K and V of a block are in registers: lane (g, c) holds dims 4 c .. (and 64 further on) of keys 4 j + g, j = 0 ..
// NL - 1; the dot products' partial sums are reduced over the lanes of a key so that lane (g, c) ends with the score of key
// 4 c + g (as the float32 models' kernel does).
template <int HD>
__device__ __forceinline__ bool relay_attend_f32(RelaySmem& sm, unsigned char* x, RelayPtr A, Watch& watch, const Step& at, int unit, int& commit_was) {
  using S = AttnF32<HD>;
  typedef float T;
  constexpr int NL = S::NL, BK = S::BK, E = S::E, KPL = S::KPL, EPL = S::EPL, PC = S::PC;
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  asm volatile("" : "+s"(A));
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int H = A->H, KVH = A->KVH, Rseq = A->Rseq, hhd = H * HD, qw = hhd + 2 * KVH * HD, l = at.l;
  const KvView kv = ldc(&A->kv);
  const RowDesc rd = ldc(&A->rd);
  const int splits = A->splits, G = H / KVH, P = G * Rseq, ppu = A->pairs, chunks = (P + ppu - 1) / ppu;
  const int split = splits - 1 - unit % splits, chunk = unit / splits % chunks, kvh = unit / (splits * chunks) % KVH, seq = unit / (splits * chunks * KVH);
  const int p0 = chunk * ppu, np = min(ppu, P - p0);
  const int c = lane & 15, g = lane >> 4;
  // keys in the cache: those before this pass's own rows
  const int len = kv.len[seq], ktot = attn_keys(kv, rd, seq);
  const int own_slot = lane < Rseq ? rd.slot[seq * Rseq + lane] : -1;  // lane r: row r's place
  int kc = ktot;
  for (int r = 0; r < Rseq; ++r) {
    const int slot = __builtin_amdgcn_readlane(own_slot, r);
    if (slot >= 0) kc = min(kc, slot);
  }
  const int blocks = (kc + BK - 1) / BK;
  const int eff = max(1, min(splits, (blocks + RELAY_BLOCKS - 1) / RELAY_BLOCKS));
  if (split >= eff) return true;
  const int64_t tok_stride = (int64_t)KVH * HD;
  const int64_t base = (int64_t)l * kv.layer_stride + (int64_t)kvh * HD + EPL * c;
  const T *const kbase = (const T*)kv.k + base, *const vbase = (const T*)kv.v + base;
  uint4 kf[NL][E], vf[NL][E];
  auto request = [&](uint4 (&to)[NL][E], const T* from, int tok) {
    each<NL>([&](auto J) {
      constexpr int j = J;
      const T* const p = from + (int64_t)of_lane<j>(tok) * tok_stride;
#pragma unroll
      for (int e = 0; e < E; ++e) to[j][e] = *(const uint4*)(p + e * 64);
    });
  };
  auto token_of = [&](int b) { return token_index(kv, seq, max(0, min(b * BK + KPL * (c & (NL - 1)) + g, kc - 1))); };
  const int first = split * RWAVES + wave;
  int tok = 0;
  if (first < blocks) {
    tok = token_of(first);
    request(kf, kbase, tok);
    request(vf, vbase, tok);
  }
  unsigned long long mask[PC];
#pragma unroll
  for (int r = 0; r < PC; ++r) {
    mask[r] = rd.mask[seq * Rseq + min(p0 + r, P - 1) % Rseq];
    pin(mask[r]);
  }
  // the own rows as keys: 16 lanes take a (row, pair), rows side by side
  const int key_row = (wave * 4 + (lane >> 4)) & (RELAY_MAX_ROWS - 1), key_pair = (wave * 4 + (lane >> 4)) / RELAY_MAX_ROWS;
  int key_seen = 0;
  if (split == 0 && key_row < Rseq && key_pair < np) {
    const int slot = rd.slot[seq * Rseq + key_row];
    key_seen = slot >= len && slot - len < 64 && ((rd.mask[seq * Rseq + (p0 + key_pair) % Rseq] >> ((slot - len) & 63)) & 1ull);
  }
  pin(key_seen);
  // this pass's queries (of the unit's pairs), keys and values
  float* const q_s = (float*)x;                 // [PC][HD]
  float* const kn = q_s + PC * HD;              // [Rseq][HD]
  float* const vn = kn + RELAY_MAX_ROWS * HD;
  float* const o_s = vn + RELAY_MAX_ROWS * HD;  // [RWAVES][PC][HD]
  {
    constexpr int MOST = 5;                     // 20 rows of up to 128: all words of a unit
    const int words = (np + 2 * Rseq) * HD, nw = (words - wave * 64 + RT - 1) / RT;
    unsigned from[MOST], to[MOST];
    const uint64_t* const qkv_words = at.words + A->mail.qkv;
#pragma unroll
    for (int i = 0; i < MOST; ++i) {            // (64 divides HD: a wave's words are of one row and head)
      const int idx = min(wave * 64 + i * RT, words - 64), item = idx / HD, e = idx % HD + lane;
      const int p = p0 + item, kr = item - np, r = item < np ? p % Rseq : kr % Rseq;
      const int col = item < np ? kvh * G + p / Rseq : (kr < Rseq ? H : H + KVH) + kvh;
      from[i] = (unsigned)((seq * Rseq + r) * qw + col * HD + e);
      const int dim = (e >> 4) * 8 + (e & 7) + ((e >> 3) & 1) * (HD >> 1);
      to[i] = (unsigned)((item < np ? item : PC + (kr < Rseq ? 0 : RELAY_MAX_ROWS) + r) * HD + dim);  // (q_s, kn and vn follow each other)
      pin(to[i]);
    }
    auto bring = [&](auto N_) {
      constexpr int N = decltype(N_)::value;
      uint64_t w[N];
      if (collect(w, [&](int i) { return qkv_words + from[i]; }, at.tag, watch, lane)) {
#pragma unroll
        for (int i = 0; i < N; ++i) q_s[to[i]] = payload(w[i]);  // (past the end the last words again)
      } else {
        sm.leave = 1;
      }
    };
    if (nw == 1) bring(std::integral_constant<int, 1>{});
    else if (nw == 2) bring(std::integral_constant<int, 2>{});
    else if (nw > 2) bring(std::integral_constant<int, MOST>{});
  }
  __syncthreads();
  if (sm.leave) return false;
  commit(watch, l, tid, commit_was);
  constexpr float scale = 1.0f / (HD == 64 ? 8.0f : 11.3137085f);
  auto exponential = [](float v) { return expf(v); };
  {
    float m_run[PC], l_run[PC], acc[PC][E * EPL];
    Query<E * EPL> q[PC];
#pragma unroll
    for (int r = 0; r < PC; ++r) {
      m_run[r] = -INFINITY;
      l_run[r] = 0.f;
#pragma unroll
      for (int i = 0; i < E * EPL; ++i) acc[r][i] = 0.f;
      if (r < np) {
#pragma unroll
        for (int e = 0; e < E; ++e) q[r].set(q_s + r * HD + e * 64 + EPL * c, e);
      }
    }
#pragma unroll 1
    for (int b = first; b < blocks; b += eff * RWAVES) {
      if (b != first) {
        tok = token_of(b);
        request(kf, kbase, tok);
        request(vf, vbase, tok);
      }
      const int key = b * BK + KPL * c + g;  // the key whose score this lane ends with (c < NL)
      float pr[PC];
#pragma unroll
      for (int r = 0; r < PC; ++r) {
        pr[r] = 0.f;
        if (r < np) {  // uniform
          float y[NL];
#pragma unroll
          for (int j = 0; j < NL; ++j) {
            y[j] = 0.f;
#pragma unroll
            for (int e = 0; e < E; ++e) y[j] = q[r].dot(kf[j][e], e, y[j]);
          }
          if constexpr (NL == 16) {
            halve_sums<8>(y, c);
          } else {
#pragma unroll
            for (int j = 0; j < NL; ++j) y[j] += row_turn<8>(y[j]);
          }
          halve_sums<4>(y, c);
          halve_sums<2>(y, c);
          halve_sums<1>(y, c);
          const bool sees = (NL == 16 || c < NL) && (key < len || (key < kc && (unsigned)(key - len) < 64u && ((mask[r] >> ((key - len) & 63)) & 1ull)));
          const float sc = sees ? y[0] * scale : -INFINITY;
          const float m_new = fmaxf(m_run[r], wave_max(sc)), m_sub = m_new == -INFINITY ? 0.f : m_new;
          pr[r] = exponential(sc - m_sub);
          if (b != first) {
            const float alpha = exponential(m_run[r] - m_sub);
            l_run[r] *= alpha;
#pragma unroll
            for (int i = 0; i < E * EPL; ++i) acc[r][i] *= alpha;
          }
          l_run[r] += pr[r];
          m_run[r] = m_new;
        }
      }
      if (b * BK + BK > kc) {  // what lies past the last key is not read into any sum
#pragma unroll
        for (int j = 0; j < NL; ++j)
          if (b * BK + KPL * j + g >= kc) {
#pragma unroll
            for (int e = 0; e < E; ++e) vf[j][e] = make_uint4(0, 0, 0, 0);
          }
      }
      each<NL>([&](auto J) {
        constexpr int j = J;
#pragma unroll
        for (int r = 0; r < PC; ++r)
          if (r < np) {
            const float pj = __int_as_float(of_lane<j>(__float_as_int(pr[r])));
#pragma unroll
            for (int e = 0; e < E; ++e)
#pragma unroll
              for (int i = 0; i < EPL; ++i) acc[r][e * EPL + i] = fmaf(pj, element(vf[j][e], i), acc[r][e * EPL + i]);
          }
      });
    }
#pragma unroll
    for (int r = 0; r < PC; ++r)
      if (r < np) {
        float lsum = 0.f;
        if (first < blocks) {
          lsum = wave_sum(l_run[r]);
#pragma unroll
          for (int i = 0; i < E * EPL; ++i) {
            float a = acc[r][i];
            acc[r][i] = xsum<32>(xsum<16>(a));
          }
          if (lane < 16) {
#pragma unroll
            for (int i = 0; i < E * EPL; i += 4)
              *(float4*)(o_s + (wave * PC + r) * HD + (i / EPL) * 64 + EPL * c + i % EPL) = make_float4(acc[r][i], acc[r][i + 1], acc[r][i + 2], acc[r][i + 3]);
          }
        }
        if (lane == 0) {
          sm.m[wave][r] = m_run[r];
          sm.l[wave][r] = lsum;
        }
      }
  }
  if (split == 0 && key_pair < PC) {
    const int c16 = lane & 15;
    const float *const a = q_s + key_pair * HD + 4 * c16, *const k = kn + key_row * HD + 4 * c16;
    float y = 0.f;
#pragma unroll
    for (int e = 0; e < HD / 64; ++e) {
      const float4 u = *(const float4*)(a + e * 64), v = *(const float4*)(k + e * 64);
      y = fmaf(u.x, v.x, fmaf(u.y, v.y, fmaf(u.z, v.z, fmaf(u.w, v.w, y))));
    }
    y += row_turn<8>(y);
    y += row_turn<4>(y);
    y += row_turn<2>(y);
    y += row_turn<1>(y);
    if (c16 == 0) sm.own[key_row][key_pair] = key_seen ? y * scale : -INFINITY;
  }
  __syncthreads();
  relay_merge<false, HD, PC>(sm, o_s, PC * HD, vn, A, watch, at, split, eff, min(RWAVES, blocks - split * RWAVES), seq, kvh, p0, np, wave, lane);
  return true;
}

// bf16 models: scores and outputs of the cached keys on the matrix cores, S = K Q^T and O^T = V^T P, at most 8 pairs.  The columns of a
// product are the pairs' hi terms (0 .. 7) and lo terms (8 .. 15) of the queries, then of the probabilities (half precision, two
// terms); a wave works on blocks of BK keys, K as it lies in the cache, V transposed out of LDS, where it is before the queries come.
template <int HD>
struct AttnBf {
  static constexpr int PC = 8;                    // most pairs of a unit
  static constexpr int BK = HD == 64 ? 64 : 32;   // keys of a block
  static constexpr int KT = BK / 16, KS = HD / 32, DB = HD / 16;
  static constexpr int QS = HD + 8, VS = HD + 16;  // rows of queries and values in LDS, padded
  static constexpr int VB = BK * VS * 2;           // bytes of a wave's values, later of its outputs [PC][HD]
  static constexpr int LDS = 2 * RELAY_MAX_ROWS * HD * 4 + PC * HD * 4 + 2 * PC * QS * 2 + RWAVES * VB;
  static_assert(VB >= PC * HD * 4, "outputs take the place of the values");
};

template <int HD>
__device__ __forceinline__ bool relay_attend_bf16(RelaySmem& sm, unsigned char* x, RelayPtr A, Watch& watch, const Step& at, int unit, int& commit_was) {
  using S = AttnBf<HD>;
  constexpr int PC = S::PC, BK = S::BK, KT = S::KT, KS = S::KS, DB = S::DB;
  constexpr int CH = HD / 8, KPL = 64 / CH, NV = BK / KPL;  // V: 16-byte chunks of a row, keys a load covers, loads
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  asm volatile("" : "+s"(A));
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), c = lane & 15, kg = lane >> 4;
  const int H = A->H, KVH = A->KVH, Rseq = A->Rseq, hhd = H * HD, qw = hhd + 2 * KVH * HD, l = at.l;
  const KvView kv = ldc(&A->kv);
  const RowDesc rd = ldc(&A->rd);
  const int splits = A->splits, G = H / KVH, P = G * Rseq, ppu = A->pairs, chunks = (P + ppu - 1) / ppu;
  const int split = splits - 1 - unit % splits, chunk = unit / splits % chunks, kvh = unit / (splits * chunks) % KVH, seq = unit / (splits * chunks * KVH);
  const int p0 = chunk * ppu, np = min(ppu, P - p0);
  // keys in the cache: those before this pass's own rows
  const int len = kv.len[seq], ktot = attn_keys(kv, rd, seq);
  const int own_slot = lane < Rseq ? rd.slot[seq * Rseq + lane] : -1;  // lane r: row r's place
  int kc = ktot;
  for (int r = 0; r < Rseq; ++r) {
    const int slot = __builtin_amdgcn_readlane(own_slot, r);
    if (slot >= 0) kc = min(kc, slot);
  }
  const int blocks = (kc + BK - 1) / BK;
  const int eff = max(1, min(splits, (blocks + RELAY_BLOCKS - 1) / RELAY_BLOCKS));
  if (split >= eff) return true;

  float* const q_s = (float*)x;                                    // [PC][HD]
  float* const kn = q_s + PC * HD;                                 // [RELAY_MAX_ROWS][HD]
  float* const vn = kn + RELAY_MAX_ROWS * HD;
  _Float16* const qh = (_Float16*)(vn + RELAY_MAX_ROWS * HD);      // [2][PC][QS]
  _Float16* const v_s = (_Float16*)((unsigned char*)(qh + 2 * PC * S::QS) + wave * S::VB);  // [BK][VS]
  const int64_t tok_stride = (int64_t)KVH * HD;
  const kv16_t* const kbase = (const kv16_t*)kv.k + (int64_t)l * kv.layer_stride + (int64_t)kvh * HD;
  const kv16_t* const vbase = (const kv16_t*)kv.v + (int64_t)l * kv.layer_stride + (int64_t)kvh * HD;
  uint4 kf[KT][KS], k2[KT][KS], v2[NV];
  auto request = [&](int b, uint4 (&k)[KT][KS]) {
    auto key = [&](int i) { return max(0, min(b * BK + i, kc - 1)); };
    int tk[KT], tv[NV];
#pragma unroll
    for (int t = 0; t < KT; ++t) tk[t] = token_index(kv, seq, key(t * 16 + c));
#pragma unroll
    for (int i = 0; i < NV; ++i) tv[i] = token_index(kv, seq, key(i * KPL + lane / CH));
#pragma unroll
    for (int t = 0; t < KT; ++t)
#pragma unroll
      for (int s = 0; s < KS; ++s) k[t][s] = *(const uint4*)(kbase + (int64_t)tk[t] * tok_stride + s * 32 + kg * 8);
#pragma unroll
    for (int i = 0; i < NV; ++i) v2[i] = *(const uint4*)(vbase + (int64_t)tv[i] * tok_stride + lane % CH * 8);
  };
  auto values_to_lds = [&](int b) {  // (what lies past the last key is not read into any sum)
    asm volatile("" ::: "memory");
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const int key = i * KPL + lane / CH;
      *(uint4*)(v_s + key * S::VS + lane % CH * 8) = b * BK + key < kc ? v2[i] : make_uint4(0, 0, 0, 0);
    }
  };
  const int first = split * RWAVES + wave, step = eff * RWAVES;
  if (first < blocks) {
    request(first, kf);
    values_to_lds(first);
    if (first + step < blocks) request(first + step, k2);
  }
  const int pair = min(c & 7, np - 1);  // this lane's pair
  unsigned long long mask = rd.mask[seq * Rseq + (p0 + pair) % Rseq];
  pin(mask);
  // the own rows as keys: 16 lanes take a (row, pair), in two turns
  int key_seen[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int item = (i * RWAVES + wave) * 4 + kg, row = item & 7, p = item >> 3;
    key_seen[i] = 0;
    if (split == 0 && row < Rseq && p < np) {
      const int slot = rd.slot[seq * Rseq + row];
      key_seen[i] = slot >= len && slot - len < 64 && ((rd.mask[seq * Rseq + (p0 + p) % Rseq] >> ((slot - len) & 63)) & 1ull);
    }
    pin(key_seen[i]);
  }
  // this pass's queries (of the unit's pairs), keys and values
  {
    constexpr int MOST = (PC + 2 * RELAY_MAX_ROWS) * HD / RT;  // all words of a unit
    const int words = (np + 2 * Rseq) * HD, nw = (words - wave * 64 + RT - 1) / RT;
    unsigned from[MOST], to[MOST];
    int half_to[MOST];
    const uint64_t* const qkv_words = at.words + A->mail.qkv;
#pragma unroll
    for (int i = 0; i < MOST; ++i) {  // (64 divides HD: a wave's words are of one row and head)
      const int idx = min(wave * 64 + i * RT, words - 64), item = idx / HD, e = idx % HD + lane;
      const int p = p0 + item, kr = item - np, r = item < np ? p % Rseq : kr % Rseq;
      const int col = item < np ? kvh * G + p / Rseq : (kr < Rseq ? H : H + KVH) + kvh;
      from[i] = (unsigned)((seq * Rseq + r) * qw + col * HD + e);
      const int dim = (e >> 4) * 8 + (e & 7) + ((e >> 3) & 1) * (HD >> 1);
      to[i] = (unsigned)((item < np ? item : PC + (kr < Rseq ? 0 : RELAY_MAX_ROWS) + r) * HD + dim);  // (q_s, kn and vn follow each other)
      half_to[i] = item < np ? item * S::QS + dim : -1;
      pin(to[i]);
      pin(half_to[i]);
    }
    auto bring = [&](auto N_) {
      constexpr int N = decltype(N_)::value;
      uint64_t w[N];
      if (collect(w, [&](int i) { return qkv_words + from[i]; }, at.tag, watch, lane)) {
#pragma unroll
        for (int i = 0; i < N; ++i) {  // (past the end the last words again)
          const float v = payload(w[i]);
          q_s[to[i]] = v;
          if (half_to[i] >= 0) {
            const _Float16 hi = (_Float16)v;
            qh[half_to[i]] = hi;
            qh[PC * S::QS + half_to[i]] = (_Float16)(v - (float)hi);
          }
        }
      } else {
        sm.leave = 1;
      }
    };
    if (nw == 1) bring(std::integral_constant<int, 1>{});
    else if (nw == 2) bring(std::integral_constant<int, 2>{});
    else if (nw > 2) bring(std::integral_constant<int, MOST>{});
  }
  __syncthreads();
  if (sm.leave) return false;
  commit(watch, l, tid, commit_was);
  constexpr float scale = ATTN_LOG2E / (HD == 64 ? 8.0f : 11.3137085f);
  float m_run = -INFINITY, l_run = 0.f;
  attn_floatx4 acc[DB];
#pragma unroll
  for (int i = 0; i < DB; ++i) acc[i] = attn_floatx4{0.f, 0.f, 0.f, 0.f};
  if (first < blocks) {
    KFrag q[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s) q[s].u = *(const uint4*)(qh + ((c >> 3) * PC + (c & 7)) * S::QS + s * 32 + kg * 8);
#pragma unroll 1
    for (int b = first;;) {
      attn_floatx4 sc[KT];
#pragma unroll
      for (int t = 0; t < KT; ++t) {
        sc[t] = attn_floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < KS; ++s) {
          KFrag k;
          k.u = kf[t][s];
          sc[t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(k.h, q[s].h, sc[t], 0, 0, 0);
        }
      }
      // lane (kg, column c): keys t * 16 + kg * 4 + e; hi and lo columns become the pair's score in both
#pragma unroll
      for (int t = 0; t < KT; ++t)
#pragma unroll
        for (int e = 0; e < 4; ++e) sc[t][e] += row_turn<8>(sc[t][e]);
      if (b * BK + BK > min(len, kc)) {  // uniform: some keys are not everybody's
#pragma unroll
        for (int t = 0; t < KT; ++t)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int key = b * BK + t * 16 + kg * 4 + e;
            const bool sees = key < kc && (key < len || (key - len < 64 && ((mask >> ((key - len) & 63)) & 1ull)));
            sc[t][e] = sees ? sc[t][e] : -INFINITY;
          }
      }
      float top = sc[0][0];
#pragma unroll
      for (int i = 1; i < KT * 4; ++i) top = fmaxf(top, sc[i >> 2][i & 3]);
      top = attn_scaled(xmax<32>(xmax<16>(top)), scale);
      const float m_new = fmaxf(m_run, top), m_sub = m_new == -INFINITY ? 0.f : m_new;
      if (b != first) {
        const float alpha = __builtin_amdgcn_exp2f(m_run - m_sub);
        l_run *= alpha;
#pragma unroll
        for (int i = 0; i < DB; ++i)
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[i][e] *= alpha;
      }
      m_run = m_new;
      half8 p[KT / 2];  // columns 0 .. 7: hi, 8 .. 15: lo terms
#pragma unroll
      for (int h = 0; h < KT / 2; ++h) {
        typedef float floatx8_t __attribute__((ext_vector_type(8)));
        floatx8_t v;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          v[e] = __builtin_amdgcn_exp2f(fmaf(sc[h * 2 + (e >> 2)][e & 3], scale, -m_sub));
          l_run += v[e];
        }
        const half8 hi = __builtin_convertvector(v, half8), lo = __builtin_convertvector(v - __builtin_convertvector(hi, floatx8_t), half8);
        p[h] = c < 8 ? hi : lo;
      }
#pragma unroll
      for (int h = 0; h < KT / 2; ++h)
#pragma unroll
        for (int i = 0; i < DB; ++i) {
          const _Float16* const at_v = v_s + (h * 32 + kg * 4 + (c >> 2)) * S::VS + i * 16 + (c & 3) * 4;
          const half4 a0 = lds_columns(at_v), a1 = lds_columns(at_v + 16 * S::VS);
          const half8 a = __builtin_shufflevector(a0, a1, 0, 1, 2, 3, 4, 5, 6, 7);
          acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a, p[h], acc[i], 0, 0, 0);
        }
      b += step;
      if (b >= blocks) break;
#pragma unroll
      for (int t = 0; t < KT; ++t)
#pragma unroll
        for (int s = 0; s < KS; ++s) kf[t][s] = k2[t][s];
      values_to_lds(b);
      if (b + step < blocks) request(b + step, k2);
    }
    l_run = xsum<32>(xsum<16>(l_run));
    // (the wave has read its values: its outputs take their place)
    float* const o = (float*)v_s;
    asm volatile("" ::: "memory");
#pragma unroll
    for (int i = 0; i < DB; ++i) {
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[i][e] += row_turn<8>(acc[i][e]);
      if (c < 8) *(attn_floatx4*)(o + c * HD + i * 16 + kg * 4) = acc[i];
    }
  }
  if (lane < PC) {
    sm.m[wave][lane] = m_run;
    sm.l[wave][lane] = l_run;
  }
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int item = (i * RWAVES + wave) * 4 + kg, row = item & 7, p = item >> 3;
    if (split == 0 && (i == 0 || np > 4)) {
      float y = 0.f;
#pragma unroll
      for (int e = 0; e < HD / 64; ++e) {
        const float4 u = *(const float4*)(q_s + p * HD + 4 * c + e * 64), v = *(const float4*)(kn + row * HD + 4 * c + e * 64);
        y = fmaf(u.x, v.x, fmaf(u.y, v.y, fmaf(u.z, v.z, fmaf(u.w, v.w, y))));
      }
      y += row_turn<8>(y);
      y += row_turn<4>(y);
      y += row_turn<2>(y);
      y += row_turn<1>(y);
      if (c == 0) sm.own[row][p] = key_seen[i] ? y * scale : -INFINITY;
    }
  }
  __syncthreads();
  relay_merge<true, HD, PC>(sm, (const float*)(qh + 2 * PC * S::QS), S::VB / 4, vn, A, watch, at, split, eff, min(RWAVES, blocks - split * RWAVES), seq, kvh, p0, np, wave, lane);
  return true;
}

// All units of workgroup `rank` of `groups`.  False: the pass goes on without what this one would have done (leave).
template <bool BF, int HD>
__device__ __forceinline__ bool relay_run(RelaySmem& sm, unsigned char* x, const RelayPtr A, Watch& watch, int rank, int groups, int& commit_was) {
  const int L = A->n_layers, slot = A->mail.slot;
  uint64_t* const words = A->mail.words + (watch.again ? (size_t)2 * slot : 0);
  int parity = 0;
  if (threadIdx.x < ROPE_SLOTS) sm.rope_unit[threadIdx.x] = -1;
  __syncthreads();
  int u0[RS_STEPS], units[RS_STEPS];  // this workgroup's first unit of each step
#pragma unroll
  for (int s = 0; s < RS_STEPS; ++s) {
    units[s] = A->units[s];
    u0[s] = ((rank - A->first[s]) % groups + groups) % groups;
  }
#pragma unroll 1
  for (int l = 0; l < L; ++l) {
    Step at;
    at.l = l;
    at.groups = groups;
    at.tag = watch.epoch << 6 | (uint32_t)(l + 1);
    at.words = words + (size_t)(l & 1) * slot;
    at.h_words = words + (size_t)(~l & 1) * slot + A->mail.hd;
#pragma unroll 1
    for (int step = 0; step < RS_STEPS; ++step) {
      const int n = step == 0 ? units[0] : step == 1 ? units[1] : step == 2 ? units[2] : step == 3 ? units[3] : units[4];
      bool fresh = true;
#pragma unroll 1
      for (int u = step == 0 ? u0[0] : step == 1 ? u0[1] : step == 2 ? u0[2] : step == 3 ? u0[3] : u0[4]; u < n; u += groups) {
        bool ok = true;
        if constexpr (BF) {
          if (step == RS_ATTN) ok = relay_attend_bf16<HD>(sm, x, A, watch, at, u, commit_was);
        } else {
          if (step == RS_ATTN) ok = relay_attend_f32<HD>(sm, x, A, watch, at, u, commit_was);
        }
        if (step != RS_ATTN) ok = relay_product<BF, HD>(sm, x, A, watch, at, step, u, fresh, parity, commit_was);
        if (!ok) return false;
        fresh = false;
      }
    }
  }
  return true;
}

template <bool BF, int HD>
__global__ __launch_bounds__(RT) __attribute__((amdgpu_waves_per_eu(2, 2))) void relay_kernel(RelayArgs args) {
  extern __shared__ __attribute__((aligned(16))) unsigned char relay_x[];
  __shared__ RelaySmem sm;
  const RelayPtr A = (RelayPtr)__builtin_amdgcn_kernarg_segment_ptr();  // (read where a value is needed, not all at the start)
  const int tid = threadIdx.x;
  Watch watch;
  watch.sync = A->sync;
  watch.status = A->status;
  watch.patience = A->patience;
  watch.give_up = A->give_up;
  watch.groups = gridDim.x;
  watch.group = blockIdx.x;
  watch.again = watch.committed = watch.settled = false;
  if (watch.group >= A->present) return;
  watch.epoch = __builtin_amdgcn_readfirstlane(*watch.sync);
  if (tid == 0) __hip_atomic_store(watch.sync + 64 + watch.group, watch.epoch * 4 + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  int commit_was = 0, rank = watch.group, groups = watch.groups;
#pragma unroll 1
  for (;;) {
    if (tid == 0) sm.leave = 0;
    __syncthreads();
    bool done = relay_run<BF, HD>(sm, relay_x, A, watch, rank, groups, commit_was);
    if (watch.again) return;
    __syncthreads();
    done = done && !sm.leave;
    __syncthreads();
    if (tid < 64) {  // what becomes of this workgroup: nothing more, unless it was counted or has left
      if (done && !watch.committed && tid == 0) commit_was = (int)__hip_atomic_exchange(watch.sync + 64 + watch.group, watch.epoch * 4, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      uint64_t word[1] = {0};
      if (!done || __builtin_amdgcn_readfirstlane(commit_was) == (int)(watch.epoch * 4 + 3)) {
        if (!done && !watch.committed) count_in(watch, tid);
        Watch w = watch;
        w.again = true;  // (a wait that ends with its word, or with the pass)
        if (!collect(word, [&](int) { return (const uint64_t*)rank_word(watch.sync, watch.group); }, watch.epoch, w, tid)) word[0] = 0xFFFFFFFFu;
      }
      if (tid == 0) sm.verdict = (uint32_t)word[0];
    }
    __syncthreads();
    const uint32_t verdict = (uint32_t)__builtin_amdgcn_readfirstlane((int)sm.verdict);
    if (!goes_on(verdict)) {
      rank = (int)(verdict & 0xFFFF);
      groups = (int)(verdict >> 16);
      if (rank == 0xFFFF) return;  // not one of those that start over, or given up
      watch.again = true;
    } else {
      // It goes on.  Whoever has left was still waiting in layer 0, or for the first time in layer 1: what it has not made all of layer 2 waits for,
      // so that layer 0's words are as they were, and its units of layer 0 once more make the same words.
      // Once: whoever leaves after that, or from beyond layer 0, does so because the pass is given up.
      if (done || watch.committed || watch.settled) return;
      watch.settled = true;
    }
  }
}

int device_cus() {
  static const int n_cus = [] {
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) cus = 0;
    return cus > 0 ? cus : 256;
  }();
  return n_cus;
}

}  // namespace

int relay_mail_words(int rows, int d, int f, int H, int KVH, int hd, int splits, RelayMail* m) {
  auto whole = [](int n) { return (n + 15) / 16 * 16; };  // lines of 16 words
  RelayMail t;
  int n = 0;
  t.words = nullptr;
  t.qkv = n; n += whole(rows * (H + 2 * KVH) * hd);
  t.att = n; n += whole(rows * H * hd);
  t.hm = n; n += whole(rows * d);
  t.act = n; n += whole(rows * f);
  t.hd = n; n += whole(rows * d);
  t.part = n; n += splits > 1 ? whole(rows * H * splits * (hd + 2)) : 0;
  t.slot = n;
  if (m) {
    t.words = m->words;
    *m = t;
  }
  return n;
}

namespace {
// Where one launch is the faster.  us of a pass of four layers, a launch a step / one launch, on 256 tokens (bf16 heads x dims, ffn):
//   12 x 64, 2048 one row 96 / 69, 5 rows 111 / 96, 8 rows 112 / 103, 8 sequences 117 / 106; 16 on 4 x 64, 4096 (29 MB a layer) 112 / 93;
//   24 x 64, 4096 (54 MB) 128 / 113; float32 4 x 64, 688 5 rows 101 / 84, 8 rows 107 / 93; 8 x 64, 1408 one row 108 / 84, 5 rows 122 / 110.
// What it saves grows with the layers, what it costs once does not; 12 x 64, 2048 of 5 rows, 2 / 12 / 24 / 48 layers: 61 / 57, 308 / 252, 604 / 486, 1193 / 948.
// Against it count the words that are handed on in a layer (everybody who needs them polls for them), those of the activation most, which all of
// down's units read; attention units (their splits are one more hand-over); units in excess of the compute units (a workgroup with units of two steps
// in a row requests the second one's weights late); more than one sequence; and, bound by their arithmetic, float32 weights.  The lines are drawn
// through 1200 shapes of 1 to 24 heads, with 1, 2, 4 and 12 layers each, contexts of 32 to 4000 tokens and 1 to 8 rows of 1 to 8 sequences, measured on
// both sides.  What they admit keeps nine tenths of what could be gained (of float32 models with heads of 64, and of one layer with heads of 128, half);
// of 2500 further passes of 2 to 24 layers eight took 1.01 to 1.03 of a launch a step, the others less.  What they leave out took up to 1.19: 8 x 128, 3264
// of 5 rows 42.5 / 47.0, 70 / 76, 359 / 382 (1, 2, 12 layers); 16 on 8 x 64, 3296 of 4 sequences, 12 layers 1.16; float32 4 on 1 x 64, 768 of 2 x 4
// rows on 2200 tokens 1.18, 1.14, 1.16 (1, 2, 4 layers).
bool relay_pays(const RelayArgs& a, int dtype, int hd, int cus) {
  const int qkv = (a.H + 2 * a.KVH) * hd, L = a.n_layers;
  const double mb = (double)((int64_t)(dtype == 1 ? 2 : 4) * ((int64_t)qkv * a.d + (int64_t)a.d * a.H * hd + (int64_t)3 * a.d * a.f)) / (1 << 20);
  const int act = a.rows * a.f, units = a.units[RS_ATTN], over = a.first[RS_GU] + a.units[RS_GU] - cus;
  const double words = (double)a.rows * (qkv + a.H * hd + 2 * a.d + a.f) / 1024;
  double against = words + 2 * act / 1024.0 + units / 10.0 + (over > 0 ? over / 20.0 : 0) + (a.B > 1 ? 4 : 0);
  if (dtype == 1) {
    const int attn = units * (hd / 64);  // (units of half as many keys at 128 dims)
    if (mb > (a.rows == 1 ? 56 : 32) || act > 16384 || attn > (act <= 6144 ? 192 : act <= 12288 ? 128 : 96)) return false;
    if (a.B == 1 && mb <= 20 && L >= (hd == 64 ? 2 : 8)) return true;  // (1.03 once, 1.02 and 1.01 of two layers, else at most 1.00)
    return against <= (hd == 64 ? (L == 1 ? 38 : L < 4 ? 47 : 52) : (L == 1 ? 17 : L < 4 ? 41 : 54));
  }
  if (mb > 16 || act > 8192 || units > (mb <= 4 ? 256 : act <= 6144 ? 128 : 64)) return false;
  against += mb;
  return against <= (hd == 64 ? (L == 1 ? 10 : L < 4 ? 34 : L < 8 ? 33 : 52) : (L == 1 ? 39 : 55));
}

int most_staged(const RelayArgs& a, int hd) {
  const int k = a.d > a.f ? a.d : a.f;
  return k > a.H * hd ? k : a.H * hd;
}
}  // namespace

int relay_plan(RelayArgs& a, int dtype, int hd, int max_context, bool any) {
  const int R = a.rows, hhd = a.H * hd, qw = (a.H + 2 * a.KVH) * hd, most = device_cus();
  if (R < 1 || R > RELAY_MAX_ROWS || a.n_layers < 1 || a.n_layers > RELAY_MAX_LAYERS || (hd != 64 && hd != 128)) return 0;
  if (a.d % 16 || a.f % 8 || most > RELAY_MAX_GROUPS || a.B * a.KVH > most || (int64_t)4 * R * most_staged(a, hd) > RELAY_MAX_LDS) return 0;
  const int N[RS_STEPS] = {qw, 0, a.d, 2 * a.f, a.d};
  // attention: bf16 units take as many pairs as there are (up to 8; the matrix cores do them side by side), float32 ones as few as give
  // every workgroup one at most; long contexts in splits
  const int heads = a.B * a.KVH, P = a.H / a.KVH * a.Rseq, pc = dtype == 1 ? 8 : hd == 64 ? 4 : 2;
  a.pairs = dtype == 1 ? (P < pc ? P : pc) : 1;
  while (a.pairs < pc && heads * ((P + a.pairs - 1) / a.pairs) > most) a.pairs *= 2;
  const int items = heads * ((P + a.pairs - 1) / a.pairs);
  const int split_keys = RELAY_BLOCKS * (hd == 128 ? 32 : 64);
  int splits = (max_context + split_keys - 1) / split_keys;
  if (splits > RELAY_MAX_SPLITS) splits = RELAY_MAX_SPLITS;
  if (splits > most / items) splits = most / items;
  if (splits < 1) splits = 1;
  a.splits = splits;
  for (int s = 0; s < RS_STEPS; ++s) {
    const int nt = N[s] / 16;
    a.strips[s] = nt > RELAY_STRIPS ? 2 : 1;
    a.units[s] = s == RS_ATTN ? items * splits : (nt + a.strips[s] - 1) / a.strips[s];
  }
  for (int s = 0; s < RS_STEPS; ++s)
    if (s != RS_ATTN && (s == RS_O ? hhd : s == RS_DOWN ? a.f : a.d) > most_terms(dtype == 1, a.strips[s])) return 0;
  // Steps that follow each other are on different workgroups as far as those suffice: whoever has no unit of a step has the next one's
  // weights, keys and addresses ready when its input comes.  o and down, which never meet, share theirs.
  const int n_mid = a.units[RS_O] > a.units[RS_DOWN] ? a.units[RS_O] : a.units[RS_DOWN];
  a.first[RS_QKV] = 0;
  a.first[RS_O] = a.first[RS_DOWN] = a.units[RS_QKV];
  a.first[RS_ATTN] = a.units[RS_QKV] + n_mid;
  a.first[RS_GU] = a.first[RS_ATTN] + a.units[RS_ATTN];
  int groups = 1;
  for (int s = 0; s < RS_STEPS; ++s) {
    const int end = a.first[s] + a.units[s];
    if (end > groups) groups = end;
  }
  if (!any && !relay_pays(a, dtype, hd, most)) return 0;
  return groups < most ? groups : most;
}

namespace {
template <bool BF, int HD>
hipError_t run_relay(const RelayArgs& a, int groups, hipStream_t s) {
  const int staged = 4 * a.rows * most_staged(a, HD), attn = BF ? AttnBf<HD>::LDS : 4 * HD * (AttnF32<HD>::PC * (1 + RWAVES) + 2 * RELAY_MAX_ROWS), lds = staged > attn ? staged : attn;
  auto kern = relay_kernel<BF, HD>;
  static std::atomic<uint64_t> ready{0};  // bit: device
  int dev = 0;
  if (const hipError_t e = hipGetDevice(&dev); e != hipSuccess) return e;
  const uint64_t bit = dev >= 0 && dev < 64 ? (uint64_t)1 << dev : 0;
  if (!(ready.load(std::memory_order_acquire) & bit)) {
    const hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, RELAY_MAX_LDS);
    if (e != hipSuccess) return e;
    ready.fetch_or(bit, std::memory_order_release);
  }
  hipLaunchKernelGGL(kern, dim3(groups), dim3(RT), lds, s, a);
  return hipGetLastError();
}
}  // namespace

hipError_t launch_relay(const RelayArgs& a, int dtype, int hd, int groups, hipStream_t s) {
  if (groups < 1 || groups > RELAY_MAX_GROUPS || a.rows > RELAY_MAX_ROWS || 4 * a.rows * most_staged(a, hd) > RELAY_MAX_LDS) return hipErrorInvalidValue;
  if (dtype == 1) return hd == 128 ? run_relay<true, 128>(a, groups, s) : run_relay<true, 64>(a, groups, s);
  return hd == 128 ? run_relay<false, 128>(a, groups, s) : run_relay<false, 64>(a, groups, s);
}

}  // namespace mtad
