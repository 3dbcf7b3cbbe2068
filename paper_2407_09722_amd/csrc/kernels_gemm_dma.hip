// Matrix products Y[R][N] = X[R][K] * W[N][K]^T for passes of many rows (a batch of token trees, Section 3.3, or a slab of
// prompt rows): the operands, packing and epilogues of the skinny kernels (kernels_gemm.hip), both operands through LDS.
//
// What bounds it.  A weight tile (16 features x 32 k) meets the hi and the lo term of every row, so a pass of R rows costs
// 4 R flops per weight element: from about 150 rows on the matrix cores take longer than the weights from HBM.  A compute
// unit's LDS moves 128 bytes per clock, reads and fills together, and feeds four matrix cores of 1024 flop per clock; what
// decides is the bytes a wave reads from LDS per matrix instruction.  So:
//   * 16 columns of the B operand are 16 rows (not 8 rows' hi and lo terms): hi and lo accumulate into the SAME registers, and
//     a wave's tile of A strips x B row groups costs A + 2B fragment reads for 2AB matrix instructions with 4AB accumulator
//     registers: 14 KiB per 48 instructions at A = 8, B = 3 (10 KiB per 24 before).
//   * fragments go from memory to LDS without passing registers (global_load_lds, 16 bytes per lane: a packed tile and an
//     activation fragment are 1 KiB contiguous, which is what one wave instruction writes), so all registers belong to the
//     tile and nothing spends issue slots on LDS writes.
//   * 8 waves: wave r of either group owns row groups r, r + 4, ..; group 0 takes the even k tiles, group 1 the odd ones, and
//     the groups run one barrier interval apart: on every SIMD one wave reads its fragments while the other issues its
//     matrix instructions.  An interval is one k tile.  k tile j lies in ring slot j % D; it is read in interval j, its slot is
//     refilled with k tile j + D in interval j + 1 (after the barrier that ends the reads), and every wave waits for its own share
//     of k tile j + 1 before the barrier that ends interval j.
//   * an activation fragment holds 8 rows, hi and lo in alternate 128-byte pieces; a B operand takes every other piece of two
//     fragments (shifting the second one by 128 bytes, so that an LDS beat touches other banks, measured the same).
//   * TALL: with more rows than a workgroup takes (prompts) and for cut reductions the groups own strips of their own and both
//     take every k tile: 256 features x 256 rows bring 48 KiB per 512 matrix instructions of a SIMD's share, against 40 KiB per
//     256.  What counts is bytes per instruction: a compute unit has about 64 KiB of requests outstanding and its loads
//     return in the order they were made, so activations that lie in L2 wait behind weights that come from HBM, and the fill
//     runs at 58 bytes per ns instead of the 140 that activations alone reach.
// Measured, us with the sums of a cut: the planned tiles and, in brackets, the best uncut ones, each product with its own epilogue, at
// 96 / 164 / 256 rows: gate/up 27648 x 5120 82 (82) / 110 (108) / 138 (136), QKV 15360 x 5120 54 (61) / 71 (80) / 85 (85), o 5120 x
// 5120 26 (34) / 34 (35) / 41 (42), down 5120 x 13824 46 (81) / 62 (88) / 77 (100); no other tiles are more than 2 % faster.  The
// kernel before this one took 122, 90, 51 and 96 at 164 rows (plain stores).  At 256 rows of the first shape (uncut, plain stores,
// 125; 1.16 PFLOP/s, hi and lo counted) the matrix instructions alone take 88 us, the activations' way to LDS 61, the weights' 60,
// launch, epilogue and barriers 24.  At 2047 rows TALL runs at 1.5 PFLOP/s while all compute units have a tile (a library product of
// 16384^3 reaches 1.58): 22016 x 4096 622 -> 537 us, 27648 x 5120 898 -> 811, 12288 x 4096 346 -> 329.
//   * MANY: side-by-side tiles of more than one a compute unit are taken by workgroups that stay (a tile's requests before the results of the
//     one before have left; the launch's arguments, row factors and ring filled once).  A workgroup a tile / workgroups that stay, us:
//     4092 rows, 11264 x 2048 309 / 287; 2047 rows, 22016 x 4096 537 / 524, 12288 x 4096 308 / 304; 2036 rows, 27648 x 5120 811 / 803, 15360 x
//     5120 451 / 450.  Of one tile a compute unit the same code is 2 % slower (2048 x 2048 71 / 72, 2048 x 5632 156 / 162): it keeps its own.
#include "common.h"
#include "gemm.h"
#include "gemm_device.h"

#include <atomic>
#include <type_traits>

namespace mtad {

namespace {

constexpr int NW = 8;                    // waves per workgroup: two groups of four
constexpr int LDS_MOST = 160 * 1024 - 1536;  // of a compute unit, less the static arrays
constexpr int PAIR = 2048;  // bytes of two activation fragments (16 rows)
constexpr int NONTEMPORAL = 2;  // cache policy operand of global_load_lds
// Weights that a single tile of rows reads (tiles of at most 64 rows, 7 or 8 strips) and that the 256 MB of last-level cache cannot
// hold from one pass to the next are requested as data that is not read again.  HBM bounds these products: 32 rows, 27648 x 5120
// 53.1 -> 48.0 us (5.9 TB/s), 32000 x 5120 61.4 -> 53.4; 64 rows, 32000 x 5120 68.7 -> 60.1.  A smaller matrix read again and again
// loses what the cache would bring (32000 x 2048 at 64 rows 24.3 -> 26.3, 57344 x 1280 32.1 -> 39.1); so do tiles of 4 to 6 strips,
// which have fewer weights on their way (22016 x 4096, 32 rows: 35.5 -> 38.2).
__host__ __device__ constexpr bool streams(int N, int K, int row_tiles) { return N >= 16384 && (int64_t)N * K >= (1 << 27) && row_tiles == 1; }

// A strips per wave; TALL: the groups own A strips each and both take every k tile, else both own the same A strips.
// B row groups of 64 rows, or B = 0: one of 32 rows (two of each group's waves hold rows, the others only bring fragments), for
// passes of 25 to 32: half the activations on their way leave room for weights in the ring (13 slots of 8 strips instead of 9) and
// among the requests.  With weights requested as above: 32000 x 5120 at 32 rows 59.1 us with a 64-row tile, 53.7 with this one.
template <int A, int B_, bool TALL>
struct DmaShape {
  static constexpr bool HALF_TILE = B_ == 0;
  static constexpr int B = HALF_TILE ? 1 : B_;       // B operands per wave
  static constexpr int XF = HALF_TILE ? 4 : 8 * B;   // activation fragments per k tile
  static constexpr int ROWS = 8 * XF;                // rows per workgroup
  static constexpr int TS = TALL ? 2 * A : A;        // strips per workgroup
  static constexpr int FRAGS = TS + XF;              // KiB that one k tile brings: weight tiles, then activation fragments
  static constexpr int LPW = (FRAGS + NW - 1) / NW;  // of them per wave
  static constexpr int FULL = FRAGS - (LPW - 1) * NW;  // waves that bring LPW; the others bring one less (HALF_TILE) or the last one again
  static constexpr bool STREAM = B_ <= 1 && A >= 7;  // may request its weights as data that is not read again
  static constexpr int SLOT = FRAGS * 1024;
  static constexpr int D0 = LDS_MOST / SLOT;
  static constexpr int D = D0 > 16 ? 16 : D0;        // ring slots
  static_assert(D >= 3, "one slot read, one arriving, one being requested");
  static constexpr int RED = TALL ? 0 : 4 * 64 * 16 * B * A;  // bytes the groups exchange
  static constexpr int LDS = D * SLOT > RED ? D * SLOT : RED;
  static_assert((D - 2) * LPW <= 63, "wait counter");
  static_assert(LDS + ROWS * 4 <= 160 * 1024, "a compute unit's LDS");
};

// s_waitcnt operand (gfx9 encoding): at most n vector memory operations outstanding, no LDS operation
constexpr int wait_vm_lds(int n) { return (n & 15) | ((n >> 4) << 14) | 0x0070; }

typedef const __attribute__((address_space(1))) uint32_t* GlobalWords;
typedef __attribute__((address_space(3))) uint32_t* LdsWords;

// ---- epilogues -----------------------------------------------------------------------------------------------------
// The values are those of gemm_epilogue (gemm_device.h); what differs is who computes and how it is stored.  A wave holds, per
// (strip, row group), features kg * 4 .. + 3 of row c in lane (kg, c), for a whole tile of strips at a time:
//   * paired strips (rotary pairs, gate and up) hold partners 32 lanes apart.  Two strips trade halves (one row-half swap per
//     register), after which lanes 0 .. 31 have both partners of the first strip and lanes 32 .. 63 those of the second.
//   * 16-bit results leave as 16 bytes per lane: lanes 16 apart hold neighbouring groups of four features; a row swap of two
//     results (hi and lo terms, or a head's first and second half) gives one lane eight features of the first and the other
//     lane eight of the second.
// With one item per (strip, row group) and 8-byte stores a tile's epilogue took 20 to 28 us of a workgroup's 180 at 2047 rows.

__device__ __forceinline__ void swap_halves(float& a, float& b) {  // a = (a's lower lanes, b's lower lanes), b = the upper ones
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  a = __uint_as_float(r[0]);
  b = __uint_as_float(r[1]);
}
// lanes of even rows (kg 0, 2): x of this lane, then x of the lane 16 further; of odd rows: y of the lane 16 before, then its own y
__device__ __forceinline__ uint4 join_rows(uint2 x, uint2 y) {
  const auto r0 = __builtin_amdgcn_permlane16_swap(x.x, y.x, false, false), r1 = __builtin_amdgcn_permlane16_swap(x.y, y.y, false, false);
  return make_uint4(r0[0], r1[0], r0[1], r1[1]);
}
__device__ __forceinline__ float sum_kg(float v) {  // over the four key groups of a row, in every lane
  auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
// two strips' results (nt and nt + 1; the second one may not exist: have2) of B row groups; rows m[j], live[j], factor inv[j]
template <int EPI, int B>
struct PairEpilogue {
  const GemmArgs& a;
  int kg;
  int m[B];
  bool live[B];
  float inv[B];
  int64_t kv_row[B];  // EPI_QKV: element offset of the row's cache slot, -1 = not stored

  __device__ __forceinline__ PairEpilogue(const GemmArgs& a_, int row0, int wr, int c, int kg_, int rows_here, const float* inv_s, bool need_kv) : a(a_), kg(kg_) {
#pragma unroll
    for (int j = 0; j < B; ++j) {
      const int mrel = (j * 4 + wr) * 16 + c;
      live[j] = mrel < rows_here;
      m[j] = row0 + min(mrel, rows_here - 1);
      inv[j] = (a.ssq && live[j]) ? inv_s[mrel] : 1.0f;
      kv_row[j] = -1;
    }
    if constexpr (EPI == EPI_QKV) {
      if (need_kv) {
#pragma unroll
        for (int j = 0; j < B; ++j) {
          const int slot = a.slot[m[j]];
          if (live[j] && slot >= 0) {
            if (slot >= kv_capacity(a.kv)) atomicOr(a.status, (uint32_t)ST_KV_CAP);
            else kv_row[j] = (int64_t)a.layer * a.kv.layer_stride + kv_token_offset(a.kv, m[j] / a.Rseq, slot);
          }
        }
      }
    }
  }
  // fragment-order address (16 bytes) of row m, features k .. k + 7 (k a multiple of 8), one plane; the pass has more than 24 rows
  __device__ __forceinline__ bf16_t* frag(bf16_t* base, int mm, int k, int plane) const {
    return base + ((((int64_t)(k >> 5) * a.ncg + (mm >> 3)) * 64 + ((k >> 3) & 3) * 16 + plane * 8 + (mm & 7)) << 3);
  }
  __device__ __forceinline__ void resid(int nt, const floatx4 (&s)[B]) const {
    const int n = nt * 16 + kg * 4;
    const float4 gn = *(const float4*)(a.g_next + n);
    float4 h[B];
#pragma unroll
    for (int j = 0; j < B; ++j) h[j] = *(const float4*)(a.h + (int64_t)m[j] * a.N + n);
#pragma unroll
    for (int j = 0; j < B; ++j) {
      const float4 hn = make_float4(h[j].x + s[j][0], h[j].y + s[j][1], h[j].z + s[j][2], h[j].w + s[j][3]);
      const float x[4] = {hn.x * gn.x, hn.y * gn.y, hn.z * gn.z, hn.w * gn.w};
      uint2 hi, lo;
      split_bf16_x4(x, hi, lo);
      const uint4 v = join_rows(hi, lo);
      const float q = sum_kg(hn.x * hn.x + hn.y * hn.y + hn.z * hn.z + hn.w * hn.w);
      if (live[j]) {
        *(float4*)(a.h + (int64_t)m[j] * a.N + n) = hn;
        *(uint4*)frag(a.planes_out, m[j], nt * 16 + (kg >> 1) * 8, kg & 1) = v;
        if (kg == 0) a.ssq_out[(int64_t)m[j] * (a.N >> 4) + nt] = q;
      }
    }
  }

  __device__ __forceinline__ void paired(int nt, floatx4 (&s)[B], floatx4 (&s2)[B], bool have2) const {
    const bool mine = kg < 2 || have2;
    const int ntl = nt + (kg >> 1);  // the strip this lane now works on
    if constexpr (EPI == EPI_SWIGLU) {
#pragma unroll
      for (int j = 0; j < B; ++j) {
        float x[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          float g = s[j][e], u = s2[j][e];
          swap_halves(g, u);
          g *= inv[j];
          u *= inv[j];
          x[e] = g / (1.0f + expf(-g)) * u;
        }
        uint2 hi, lo;
        split_bf16_x4(x, hi, lo);
        const uint4 v = join_rows(hi, lo);
        if (live[j] && mine) *(uint4*)frag(a.act_out, m[j], ntl * 8, kg & 1) = v;
      }
    } else {  // EPI_QKV
      typedef kv16_t half4_t __attribute__((ext_vector_type(4)));
      const int hd = a.kv.head_dim, half = hd >> 1, tph = hd >> 4, H = a.n_heads, KVH = a.kv.n_kv_heads;
      const int head = ntl / tph, i8 = (ntl % tph) * 8, i = i8 + (kg & 1) * 4;
      const bool turned = mine && head < H + KVH;  // q and k heads are rotated
      float4 cs[B][2];
#pragma unroll
      for (int j = 0; j < B; ++j) {
        cs[j][0] = cs[j][1] = make_float4(1.f, 0.f, 1.f, 0.f);
        if (turned) {
          const float4* t = (const float4*)(a.rope + (int64_t)m[j] * half + i);
          cs[j][0] = t[0];
          cs[j][1] = t[1];
        }
      }
#pragma unroll
      for (int j = 0; j < B; ++j) {
        float x1[4], x2[4];
        const float co[4] = {cs[j][0].x, cs[j][0].z, cs[j][1].x, cs[j][1].z}, si[4] = {cs[j][0].y, cs[j][0].w, cs[j][1].y, cs[j][1].w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          float p = s[j][e], r = s2[j][e];
          swap_halves(p, r);
          p *= inv[j];
          r *= inv[j];
          x1[e] = turned ? p * co[e] - r * si[e] : p;
          x2[e] = turned ? r * co[e] + p * si[e] : r;
        }
        half4_t v1, v2;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          v1[e] = (kv16_t)x1[e];
          v2[e] = (kv16_t)x2[e];
        }
        const uint4 v = join_rows(*(uint2*)&v1, *(uint2*)&v2);
        if (!live[j] || !mine) continue;
        if (head < H) {
          float* const q = a.q_out + (int64_t)m[j] * H * hd + head * hd + i;
          *(float4*)q = make_float4(x1[0], x1[1], x1[2], x1[3]);
          *(float4*)(q + half) = make_float4(x2[0], x2[1], x2[2], x2[3]);
        } else if (kv_row[j] >= 0) {
          const bool is_k = head < H + KVH;
          const int gh = head - (is_k ? H : H + KVH);
          *(uint4*)((kv16_t*)(is_k ? a.kv.k : a.kv.v) + kv_row[j] + gh * hd + (kg & 1) * half + i8) = v;
        }
      }
    }
  }
};

// the kernel's first argument, to be read from memory again
__device__ __forceinline__ const GemmArgs& fresh_args() {
  const __attribute__((address_space(4))) GemmArgs* p = (const __attribute__((address_space(4))) GemmArgs*)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return *(const GemmArgs*)p;
}

template <int A, int B_, bool TALL, bool MANY, int EPI>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(2, 2))) void gemm_bf16_dma_kernel(GemmArgs args, int tiles_n, int tiles_m, int KS) {
  using Sh = DmaShape<A, B_, TALL>;
  constexpr int B = Sh::B, LPW = Sh::LPW, D = Sh::D, SLOT = Sh::SLOT, TS = Sh::TS;
  extern __shared__ __attribute__((aligned(16))) unsigned char lds_dma[];
  __shared__ float inv_s[Sh::ROWS];
  const GemmArgs& a = args;
  // (what the first requests need of the arguments at once; left to itself the compiler fetches it in three rounds, each a trip to memory)
  asm volatile("" ::"s"(a.W), "s"(a.X), "s"(a.R), "s"(a.N), "s"(a.K), "s"(a.ncg), "s"(a.ssq), "s"(a.NP), "s"(tiles_n), "s"(tiles_m), "s"(KS));

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wr = wave & 3, grp = wave >> 2;
  const bool rowless = Sh::HALF_TILE && wr >= 2;  // waves that only bring fragments
  const bool full = !Sh::HALF_TILE || wave < Sh::FULL;
  const bool stream = Sh::STREAM && streams(a.N, a.K, tiles_m);
  const int c = lane & 15, kg = lane >> 4;
  const int KT_all = a.K >> 5, NT = a.N >> 4;
  // workgroups go to the 8 XCDs in turn: give each XCD a contiguous range of tiles, and within it blocks of up to four row tiles
  // by a few feature tiles, so that its L2 serves a weight tile to four workgroups and an activation fragment to several
  const int tiles = tiles_n * tiles_m, total = tiles * KS, per = (KT_all + KS - 1) / KS;
  struct Tile {
    int nt0, row0, ks, k_lo, n_kt;
  };
  auto place = [&](int id) {
    const int xcd = id & 7;
    int l = xcd * (total >> 3) + min(xcd, total & 7) + (id >> 3);
    const int ks = l / tiles;
    l -= ks * tiles;
    const int per_group = 4 * tiles_n, mg = l / per_group, lg = l - mg * per_group;
    const int gm = min(4, tiles_m - mg * 4);
    const int tm = mg * 4 + lg % gm, tn = lg / gm;
    const int k_lo = ks * per;
    return Tile{tn * TS, tm * Sh::ROWS, ks, k_lo, min(KT_all, k_lo + per) - k_lo};  // the launcher leaves no range empty
  };

  // What this wave requests per k tile: fragment f = i * 8 + wave is weight tile f, or activation fragment f - TS; those past
  // the last one read it again, to the same place with the same contents (32-row tiles leave them out).  (Weights on waves of
  // their own, requested much earlier than the activations, were no faster: a compute unit's loads return in the order of their
  // requests, so the activations behind them wait for HBM all the same, and the ring holds fewer of them.)
  const char* src[LPW];
  size_t step[LPW];
  unsigned dst[LPW];
  int s_in = 0;  // ring slot of the next request, in bytes
  auto aim = [&](const Tile& at) {
    const int cg0 = at.row0 >> 3, cg_last = a.ncg - 1;
#pragma unroll
    for (int i = 0; i < LPW; ++i) {
      const int f = min(i * NW + wave, Sh::FRAGS - 1);
      if (f < TS) {
        src[i] = (const char*)a.W + (((size_t)min(at.nt0 + f, NT - 1) * KT_all + at.k_lo) << 10);
        step[i] = 1024;
        dst[i] = (unsigned)f * 1024u;
      } else {
        const int x = f - TS;
        src[i] = (const char*)a.X + (((size_t)at.k_lo * a.ncg + min(cg0 + x, cg_last)) << 10);
        step[i] = (size_t)a.ncg << 10;
        dst[i] = (unsigned)f * 1024u;
      }
    }
    s_in = 0;
  };
  auto request = [&](auto FROM, auto TO) {  // its share of a k tile, or part of it; the slot moves on with the last part
#pragma unroll
    for (int i = FROM; i < TO; ++i) {
      if (i == LPW - 1 && !full) break;
      if (stream && i * NW + wave < TS)
        __builtin_amdgcn_global_load_lds((GlobalWords)(src[i] + (unsigned)lane * 16u), (LdsWords)(lds_dma + s_in + dst[i]), 16, 0, NONTEMPORAL);
      else
        __builtin_amdgcn_global_load_lds((GlobalWords)(src[i] + (unsigned)lane * 16u), (LdsWords)(lds_dma + s_in + dst[i]), 16, 0, 0);
      src[i] += step[i];
      // Side-by-side tiles: the address moves on where it is.  Left to itself the compiler computes those of two requests ahead of both and copies them
      // back, three to five more scalar instructions a k tile, between a barrier and the requests.
      if constexpr (TALL) {
        asm volatile("" : "+s"(src[i]));
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    if constexpr (TO == LPW) s_in = s_in + SLOT == D * SLOT ? 0 : s_in + SLOT;
  };
  constexpr std::integral_constant<int, 0> NONE{};
  constexpr std::integral_constant<int, LPW / 2> HALF{};
  constexpr std::integral_constant<int, LPW> ALL{};
  constexpr int ahead = D - 1;
  auto row_factors = [&](int row0) {
    GemmArgs ar = MANY ? fresh_args() : a;
    ar.row0 = row0;
    gemm_row_factors<false, 8>(ar, inv_s, min(Sh::ROWS, a.R - row0), wave, lane, NW);
  };
  int id = (int)blockIdx.x;
  Tile at = place(id);
  aim(at);
  for (int j = 0; j < ahead && j < at.n_kt; ++j) request(NONE, ALL);
  row_factors(at.row0);

  floatx4 acc[A][B];
  // lane (kg, row) of a B operand: fragment row / 8 of the pair, piece (kg, plane), row % 8
  const unsigned w_off = (unsigned)((TALL ? grp * A * 1024 : 0) + lane * 16);
  const unsigned x_off = (unsigned)(TS * 1024 + (Sh::HALF_TILE ? wr & 1 : wr) * PAIR + (c >> 3) * 1024 + (kg * 16 + (c & 7)) * 16);
  Frag fw[A], fx[B][2];
  constexpr int STRIDE = TALL ? SLOT : 2 * SLOT;
  int s_out;  // ring slot of this group's next k tile
  auto fetch = [&]() {
    const unsigned char *const wp = lds_dma + s_out + w_off, *const xp = lds_dma + s_out + x_off;
#pragma unroll
    for (int si = 0; si < A; ++si) fw[si].n = *(const uintx4*)(wp + si * 1024);
#pragma unroll
    for (int j = 0; j < B; ++j) {
      fx[j][0].n = *(const uintx4*)(xp + j * (4 * PAIR));
      fx[j][1].n = *(const uintx4*)(xp + j * (4 * PAIR) + 128);
    }
    s_out += STRIDE;
    if (s_out >= D * SLOT) s_out -= D * SLOT;
  };
  // An interval ends: this wave's requests for the next k tile have arrived (all but its requests for later ones, or all
  // of them when it has no more to make), its fragment reads are done, then the barrier.  The fences keep the compiler
  // from moving memory operations across (the barrier alone does not).
  auto interval_end = [&](bool steady) {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
    if (steady && full) __builtin_amdgcn_s_waitcnt(wait_vm_lds((D - 2) * LPW));
    else if (steady) __builtin_amdgcn_s_waitcnt(wait_vm_lds((D - 2) * (LPW - 1)));
    else __builtin_amdgcn_s_waitcnt(wait_vm_lds(0));
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };

  auto barrier = [&]() {  // an interval after which nothing new has to have arrived
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(wait_vm_lds(63));
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  auto multiply = [&]() {
#pragma unroll
    for (int j = 0; j < B; ++j)
#pragma unroll
      for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int si = 0; si < A; ++si) acc[si][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fw[si].v, fx[j][p].v, acc[si][j], 0, 0, 0);
  };

  // MANY: the launch has one workgroup a compute unit, which works on tiles id, id + workgroups, .. (the count is a multiple of 8, so it stays in
  // its XCD's range).  The ring is free after a tile's last barrier: the next tile's first k tiles arrive while this one's results
  // leave, and workgroups drift apart, so that one's results leave under another's matrix instructions.
#pragma unroll 1
  for (bool first = true;; first = false) {
    const int n_kt = at.n_kt, nt0 = at.nt0, row0 = at.row0;
    s_out = TALL ? 0 : grp * SLOT;
#pragma unroll
    for (int si = 0; si < A; ++si)
#pragma unroll
      for (int j = 0; j < B; ++j) acc[si][j] = floatx4{0.f, 0.f, 0.f, 0.f};
    interval_end(first && n_kt >= ahead);  // k tile 0 is there (and the row factors); later ones: all requested, whatever the results' stores count
    if constexpr (!TALL) {
      int i = 0;  // interval: k tile i + ahead is requested in it
      if (grp == 1) {
        const bool more = i + ahead < n_kt;
        if (more) request(NONE, ALL);
        interval_end(more);
        ++i;
      }
      const int trips = (n_kt + 1) >> 1;
#pragma unroll 1
      for (int t = 0; t < trips; ++t) {
        {  // memory interval: fragments of this group's k tile
          const bool more = i + ahead < n_kt;
          if (!rowless) fetch();
          if (more) request(NONE, ALL);
          interval_end(more);
          ++i;
        }
        {  // compute interval
          const bool more = i + ahead < n_kt;
          if (more) request(NONE, ALL);
          __builtin_amdgcn_sched_barrier(0);
          if (!rowless && (grp == 0 || 2 * t + 1 < n_kt)) multiply();
          interval_end(more);
          ++i;
        }
      }
      if (grp == 0) interval_end(false);
    } else {
      // two intervals per k tile: group 0 reads k tile j in interval 2j and multiplies in 2j + 1, group 1 one interval later; k tile
      // j + ahead goes out in halves in the same two intervals (its slot was last read in interval 2j - 1), and k tile j + 1 has
      // arrived at the end of 2j + 1
      if (grp == 0) {
#pragma unroll 1
        for (int j = 0; j < n_kt; ++j) {
          const bool more = j + ahead < n_kt;
          fetch();
          if (more) request(NONE, HALF);
          barrier();
          if (more) request(HALF, ALL);
          __builtin_amdgcn_sched_barrier(0);
          multiply();
          interval_end(more);
        }
        barrier();
      } else {
        if (ahead < n_kt) request(NONE, HALF);
        barrier();
#pragma unroll 1
        for (int j = 0; j < n_kt; ++j) {
          const bool more = j + ahead < n_kt;
          fetch();
          if (more) request(HALF, ALL);
          interval_end(more);
          if (j + 1 + ahead < n_kt) request(NONE, HALF);
          __builtin_amdgcn_sched_barrier(0);
          multiply();
          barrier();
        }
      }
    }

    // (the arguments that the results' way out reads; held across the tiles they cost 20 to 70 more scalar spills)
    const GemmArgs& a = MANY ? fresh_args() : args;
    const int next_id = id + (int)gridDim.x;
    const bool again = MANY && next_id < total;
    Tile next = at;
    if (again) {
      next = place(next_id);
      aim(next);
      for (int j = 0; j < ahead && j < next.n_kt; ++j) request(NONE, ALL);
    }

    // not TALL: the groups' sums meet in LDS; group 0 finishes the first half of the pairs of strips, group 1 the others
    constexpr int PAIRS = (A + 1) / 2, PH = (PAIRS + 1) / 2;
    floatx4* const red = reinterpret_cast<floatx4*>(lds_dma);  // [4 waves][A][B][64]
    auto owns = [&](int p) { return TALL || (p < PH) == (grp == 0); };
    if constexpr (!TALL) {
#pragma unroll
      for (int si = 0; si < A; ++si)
        if (!owns(si >> 1)) {
#pragma unroll
          for (int j = 0; j < B; ++j) red[((wr * A + si) * B + j) * 64 + lane] = acc[si][j];
        }
      __syncthreads();
#pragma unroll
      for (int si = 0; si < A; ++si)
        if (owns(si >> 1)) {
#pragma unroll
          for (int j = 0; j < B; ++j) {
            const floatx4 o = red[((wr * A + si) * B + j) * 64 + lane];
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[si][j][e] += o[e];
          }
        }
    }
    const int rows_here = min(Sh::ROWS, a.R - row0);
    const int nt_wave = nt0 + (TALL ? grp * A : 0);
    const bool need_kv = EPI == EPI_QKV && KS == 1 && (nt_wave + A) * 16 > a.n_heads * a.kv.head_dim;
    const PairEpilogue<EPI, B> fin(a, row0, wr, c, kg, rows_here, inv_s, need_kv);
#pragma unroll
    for (int p = 0; p < PAIRS; ++p) {
      constexpr int LAST = A - 1;
      const int nt = nt_wave + 2 * p;
      if (!owns(p) || nt >= NT || rowless) continue;
      const bool have2 = 2 * p + 1 < A && nt + 1 < NT;
      if (KS > 1) {  // the launch after this one adds the ranges: part[range][row][packed feature]
#pragma unroll
        for (int o = 0; o < 2; ++o)
          if (o == 0 || have2) {
#pragma unroll
            for (int j = 0; j < B; ++j)
              if (fin.live[j]) *(floatx4*)(a.part + ((size_t)at.ks * a.R + fin.m[j]) * a.N + (nt + o) * 16 + kg * 4) = acc[2 * p + o < A ? 2 * p + o : LAST][j];
          }
      } else if constexpr (EPI == EPI_SWIGLU || EPI == EPI_QKV) {
        fin.paired(nt, acc[2 * p], acc[2 * p + 1 < A ? 2 * p + 1 : LAST], have2);
      } else {
#pragma unroll
        for (int o = 0; o < 2; ++o)
          if (o == 0 || have2) {
            floatx4 (&s)[B] = acc[2 * p + o < A ? 2 * p + o : LAST];
            if constexpr (EPI == EPI_RESID) {
              fin.resid(nt + o, s);
            } else {
#pragma unroll
              for (int j = 0; j < B; ++j) gemm_epilogue<EPI>(a, nt + o, s[j], fin.m[j], fin.live[j], fin.inv[j], kg);
            }
          }
      }
    }
    if (!again) break;
    if (next.row0 != row0) {
      __syncthreads();  // the factors of this tile have been read
      row_factors(next.row0);
    }
    id = next_id;
    at = next;
  }
}

// After a product whose reduction dimension was cut into KS ranges: grid (pieces of ROW_PIECE features, rows), every workgroup adds the
// ranges of its piece in order.
//   RESID  the residual epilogue: h += sum, the next norm's input h * gain as hi / lo terms, and the sum of squares of the piece, so
//          that the products that read them have a handful of values per row left to add
//   STORE  the piece of Y
// Bound by the ranges' way from memory; a workgroup per row (164 rows x 5120, 8 ranges, 27 MB: 11.9 us) left compute units idle, 10.7; 40 rows x 4096 (21 MB) 6.2, 5.0.
constexpr int RT = 256, ROW_PIECE = RT * 4;
template <int KS, int EPI>
__global__ __launch_bounds__(RT) void gemm_rows_kernel(GemmArgs a) {
  __shared__ float sh[RT / 64];
  const int m = blockIdx.y, N = a.N, n = blockIdx.x * ROW_PIECE + (int)threadIdx.x * 4;
  const size_t range = (size_t)a.R * N;
  float q = 0.f;
  if (n < N) {
    const float* const p = a.part + (size_t)m * N + n;
    float4 t[KS];
#pragma unroll
    for (int k = 0; k < KS; ++k) t[k] = *(const float4*)(p + k * range);
    float4 o = make_float4(0.f, 0.f, 0.f, 0.f), gn = o;
    if constexpr (EPI == EPI_RESID) {
      o = *(const float4*)(a.h + (int64_t)m * N + n);
      gn = *(const float4*)(a.g_next + n);
    }
    float4 s = t[0];
#pragma unroll
    for (int k = 1; k < KS; ++k) { s.x += t[k].x; s.y += t[k].y; s.z += t[k].z; s.w += t[k].w; }
    if constexpr (EPI == EPI_STORE) {
      float4* const y = (float4*)(a.Y + (int64_t)m * a.ldy + n);
      if (a.accumulate) {
        o = *y;
        s.x += o.x; s.y += o.y; s.z += o.z; s.w += o.w;
      }
      *y = s;
    } else {
      s.x += o.x; s.y += o.y; s.z += o.z; s.w += o.w;
      *(float4*)(a.h + (int64_t)m * N + n) = s;
      const float x[4] = {s.x * gn.x, s.y * gn.y, s.z * gn.z, s.w * gn.w};
      uint2 hi, lo;
      split_bf16_x4(x, hi, lo);
      *(uint2*)(a.planes_out + act_offset(a.ncg, a.R, N, 0, m, n)) = hi;
      *(uint2*)(a.planes_out + act_offset(a.ncg, a.R, N, 1, m, n)) = lo;
      q = s.x * s.x + s.y * s.y + s.z * s.z + s.w * s.w;
    }
  }
  if constexpr (EPI == EPI_RESID) {
    q = wave_sum(q);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = q;
    __syncthreads();
    if (threadIdx.x == 0) {
      for (int w = 1; w < RT / 64; ++w) q += sh[w];
      a.ssq_out[(int64_t)m * gridDim.x + blockIdx.x] = q;
    }
  }
}

// The same for products whose strips hold partners 8 features apart (rotary pairs, gate and up): one thread per (row, strip,
// four pairs), grid (quads of the row, rows).
template <int KS, int EPI>
__global__ __launch_bounds__(256) void gemm_pairs_kernel(GemmArgs a) {
  const int m = blockIdx.y, lane = threadIdx.x & 63, NT = a.N >> 4;
  float inv = 1.0f;
  if (a.ssq) {
    float s = 0.f;
    for (int p = lane; p < a.NP; p += 64) s += a.ssq[(int64_t)m * a.NP + p];
    s = wave_sum(s);
    inv = 1.0f / sqrtf(s / (float)a.K + a.eps);
  }
  const int item = blockIdx.x * 256 + threadIdx.x, nt = item >> 1, i0 = (item & 1) * 4;
  if (nt >= NT) return;
  const float* const p = a.part + (size_t)m * a.N + nt * 16 + i0;
  const size_t range = (size_t)a.R * a.N;
  float4 t1[KS], t2[KS];
#pragma unroll
  for (int k = 0; k < KS; ++k) {
    t1[k] = *(const float4*)(p + k * range);
    t2[k] = *(const float4*)(p + k * range + 8);
  }
  float4 s1 = t1[0], s2 = t2[0];
#pragma unroll
  for (int k = 1; k < KS; ++k) {
    s1.x += t1[k].x; s1.y += t1[k].y; s1.z += t1[k].z; s1.w += t1[k].w;
    s2.x += t2[k].x; s2.y += t2[k].y; s2.z += t2[k].z; s2.w += t2[k].w;
  }
  float x1[4] = {s1.x * inv, s1.y * inv, s1.z * inv, s1.w * inv}, x2[4] = {s2.x * inv, s2.y * inv, s2.z * inv, s2.w * inv};
  if constexpr (EPI == EPI_SWIGLU) {
    float x[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) x[e] = x1[e] / (1.0f + expf(-x1[e])) * x2[e];
    uint2 hi, lo;
    split_bf16_x4(x, hi, lo);
    *(uint2*)(a.act_out + act_offset(a.ncg, a.R, a.N >> 1, 0, m, nt * 8 + i0)) = hi;
    *(uint2*)(a.act_out + act_offset(a.ncg, a.R, a.N >> 1, 1, m, nt * 8 + i0)) = lo;
  } else {
    const int hd = a.kv.head_dim, half = hd >> 1, tph = hd >> 4, H = a.n_heads, KVH = a.kv.n_kv_heads;
    const int head = nt / tph, i = (nt % tph) * 8 + i0;
    if (head < H + KVH) {  // q and k heads are rotated
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float2 cs = a.rope[(int64_t)m * half + i + e];
        const float y1 = x1[e] * cs.x - x2[e] * cs.y, y2 = x2[e] * cs.x + x1[e] * cs.y;
        x1[e] = y1;
        x2[e] = y2;
      }
    }
    if (head < H) {
      float* const q = a.q_out + (int64_t)m * H * hd + head * hd + i;
      *(float4*)q = make_float4(x1[0], x1[1], x1[2], x1[3]);
      *(float4*)(q + half) = make_float4(x2[0], x2[1], x2[2], x2[3]);
    } else {
      const int slot = a.slot[m];
      if (slot < 0) return;
      if (slot >= kv_capacity(a.kv)) {
        atomicOr(a.status, (uint32_t)ST_KV_CAP);
        return;
      }
      typedef kv16_t half4_t __attribute__((ext_vector_type(4)));
      half4_t v1, v2;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        v1[e] = (kv16_t)x1[e];
        v2[e] = (kv16_t)x2[e];
      }
      const bool is_k = head < H + KVH;
      kv16_t* const dst = (kv16_t*)(is_k ? a.kv.k : a.kv.v) + (int64_t)a.layer * a.kv.layer_stride + kv_token_offset(a.kv, m / a.Rseq, slot) +
                          (head - (is_k ? H : H + KVH)) * hd + i;
      *(uint2*)dst = *(uint2*)&v1;
      *(uint2*)(dst + half) = *(uint2*)&v2;
    }
  }
}

// Activation planes [2][R][K] -> fragments (act_offset's order for more than 24 rows); rows past R are zeros.  One wave per
// fragment.
__global__ __launch_bounds__(256) void xfrag_kernel(const bf16_t* __restrict__ X, bf16_t* __restrict__ out, int R, int K, int ncg) {
  const int lane = threadIdx.x & 63;
  const int64_t f = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (f >= (int64_t)(K >> 5) * ncg) return;
  const int kt = (int)(f / ncg), cg = (int)(f % ncg);
  const int row = cg * 8 + (lane & 7), plane = (lane >> 3) & 1;
  uint4 v = make_uint4(0, 0, 0, 0);
  if (row < R) v = *(const uint4*)(X + ((size_t)plane * R + row) * K + kt * 32 + (lane >> 4) * 8);
  *(uint4*)(out + (f * 64 + lane) * 8) = v;
}

int device_cus() {
  static const int n_cus = [] {
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) cus = 0;
    return cus > 0 ? cus : 256;
  }();
  return n_cus;
}

// workgroups of a launch whose workgroups take several tiles each: one a compute unit, as many on every XCD
int resident_groups() { return device_cus() & ~7; }

struct Plan {
  int A, B, KS, tiles_n, tiles_m;
  bool tall;
  int lds = 0;  // bytes a compute unit is taken to have; 0: ask the device
};

// LDS of one compute unit of the device (the most a workgroup can be given); 160 KiB on gfx950 if the query fails
int device_lds_bytes(int dev) {
  int v = 0;
  if (hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerMultiprocessor, dev) != hipSuccess) v = 0;
  return v > 0 ? v : 160 * 1024;
}
constexpr int KS_MAX = 8;
// partial sums per range must add up to the whole product, and what reads them (run_sum) knows neither row factors nor logsumexps
bool can_cut(const GemmArgs& a, int epi) { return a.part && !(epi == EPI_STORE && (a.lse_part || a.ssq)); }
bool cut_fits(const GemmArgs& a, int KS) {
  const int KT = a.K >> 5, per = (KT + KS - 1) / KS;
  return KS <= KS_MAX && per * (KS - 1) < KT /* no range is empty */ && (size_t)KS * a.R * a.N <= a.part_floats;
}

// Rows per workgroup (32, or 64 to 256), strips per workgroup (4 to 8, or 10 to 16 with the groups side by side where 129 rows and more
// meet) and ranges of the reduction dimension: the cheapest by a count of clocks per compute unit.  A k tile lasts as long as its
// matrix instructions, its LDS traffic, its way to LDS (about 25 bytes per clock where weights from HBM and activations from L2
// alternate) or its weights from HBM (10 to 11 bytes per clock and compute unit), plus the barriers.  A cut costs its partial
// sums' way through memory and a launch.
Plan plan_for(const GemmArgs& a, int epi) {
  Plan best{};
  const int NT = a.N >> 4, KT = a.K >> 5, cus = device_cus();
  const bool cuts = can_cut(a, epi);
  double best_cost = 0;
  for (int B_ = 4; B_ >= 0; --B_) {
    const int B = B_ ? B_ : 1, rows = B_ ? 64 * B_ : 32, tm = (a.R + rows - 1) / rows;
    if (B_ == 0 ? tm > 1 : a.R <= 32) continue;                               // up to 32 rows: a tile of 32
    if (B_ > 1 && (a.R + 64 * (B - 1) - 1) / (64 * (B - 1)) == tm) continue;  // as many tiles of fewer rows
    for (int TS : {16, 14, 12, 10, 8, 7, 6, 5, 4}) {
      const bool tall = TS > 8;
      if (tall ? B_ < 3 : TS == 4 && B_ > 1) continue;  // (4 strips meet more than 64 rows in no plan at 256 compute units)
      const int tn = (NT + TS - 1) / TS, frags = TS + rows / 8;
      const int mfma = 32 * TS * B, lds = 32 * (tall ? TS + 4 * B : TS + 2 * B) + 8 * frags, fill = 40 * frags;
      const int hbm = (B_ <= 1 && TS >= 7 && streams(a.N, a.K, tm) ? 90 : 98) * TS / tm;
      int interval = mfma;
      for (int x : {lds, fill, hbm}) interval = x > interval ? x : interval;
      interval += tall ? 250 : 100;
      for (int KS = 1; KS <= KS_MAX; ++KS) {
        const int total = tn * tm * KS;
        if (KS > 1) {
          if (!cuts || total > cus || KT < 16 * KS) break;
          if (!cut_fits(a, KS)) continue;
        }
        const int rounds = (total + cus - 1) / cus;
        double cost = (double)rounds * (((KT + KS - 1) / KS) * (double)interval + 8000);
        if (KS > 1) cost = 1.08 * (cost + 6000 + (double)(2 * KS) * a.R * a.N * 4 / 2000);  // worth it when clearly better
        if (best.A == 0 || cost < best_cost) {
          best_cost = cost;
          best = Plan{tall ? TS / 2 : TS, B_, KS, tn, tm, tall};
        }
      }
    }
  }
  return best;
}

Plan plan_of(const GemmArgs& a, const GemmTiles& t) {
  const int TS = t.strips << t.tall, NT = a.N >> 4;
  const int rows = t.row_groups ? 64 * t.row_groups : 32;
  return Plan{t.strips, t.row_groups, t.ranges, (NT + TS - 1) / TS, (a.R + rows - 1) / rows, t.tall != 0, t.lds};
}

template <int A, int B, bool TALL, bool MANY, int EPI>
hipError_t run_launch(const GemmArgs& a, const Plan& p, hipStream_t s) {
  using Sh = DmaShape<A, B, TALL>;
  auto kern = gemm_bf16_dma_kernel<A, B, TALL, MANY, EPI>;
  // Once per device: its compute units hold the ring, and more than 64 KiB of dynamic LDS needs the attribute.  A success is
  // remembered (bit d: device d; beyond 63 every launch asks), a failure is reported and tried again.
  static std::atomic<uint64_t> ready{0};
  int dev = 0;
  if (const hipError_t e = hipGetDevice(&dev); e != hipSuccess) return e;
  const uint64_t bit = dev >= 0 && dev < 64 ? (uint64_t)1 << dev : 0;
  if (p.lds || !(ready.load(std::memory_order_acquire) & bit)) {
    constexpr int STATIC = (int)sizeof(float) * Sh::ROWS;  // the kernel's own array
    if (Sh::LDS + STATIC > (p.lds ? p.lds : device_lds_bytes(dev))) return hipErrorInvalidValue;
    const hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, Sh::LDS);
    if (e != hipSuccess) return e;
    ready.fetch_or(bit, std::memory_order_release);
  }
  hipLaunchKernelGGL(kern, dim3((unsigned)(MANY ? resident_groups() : p.tiles_n * p.tiles_m * p.KS)), dim3(NW * 64), Sh::LDS, s, a, p.tiles_n, p.tiles_m, p.KS);
  return hipGetLastError();
}

template <int A, int B, bool TALL, int EPI>
hipError_t run_shape(const GemmArgs& a, const Plan& p, hipStream_t s) {
  if constexpr (TALL) {
    if (resident_groups() && p.tiles_n * p.tiles_m * p.KS > resident_groups()) return run_launch<A, B, TALL, true, EPI>(a, p, s);
  }
  return run_launch<A, B, TALL, false, EPI>(a, p, s);
}

template <int A, int EPI>
hipError_t run_rows(const GemmArgs& a, const Plan& p, hipStream_t s) {
  switch (p.B) {
    case 0: return run_shape<A, 0, false, EPI>(a, p, s);
    case 1: return run_shape<A, 1, false, EPI>(a, p, s);
  }
  if constexpr (A > 4) switch (p.B) {
    case 2: return run_shape<A, 2, false, EPI>(a, p, s);
    case 3: return run_shape<A, 3, false, EPI>(a, p, s);
    case 4: return run_shape<A, 4, false, EPI>(a, p, s);
  }
  return hipErrorInvalidValue;
}

template <int A, int EPI>
hipError_t run_tall(const GemmArgs& a, const Plan& p, hipStream_t s) {
  return p.B == 4 ? run_shape<A, 4, true, EPI>(a, p, s) : run_shape<A, 3, true, EPI>(a, p, s);
}

int row_pieces(int N) { return (N + ROW_PIECE - 1) / ROW_PIECE; }  // never more than there are strips

template <int KS, int EPI>
hipError_t run_sum_ks(const GemmArgs& a, hipStream_t s) {
  if constexpr (EPI == EPI_SWIGLU || EPI == EPI_QKV)
    hipLaunchKernelGGL((gemm_pairs_kernel<KS, EPI>), dim3((unsigned)((a.N / 8 + 255) / 256), (unsigned)a.R), dim3(256), 0, s, a);
  else
    hipLaunchKernelGGL((gemm_rows_kernel<KS, EPI>), dim3((unsigned)row_pieces(a.N), (unsigned)a.R), dim3(RT), 0, s, a);
  return hipGetLastError();
}
template <int EPI>
hipError_t run_sum(const GemmArgs& a, int KS, hipStream_t s) {
  switch (KS) {
    case 2: return run_sum_ks<2, EPI>(a, s);
    case 3: return run_sum_ks<3, EPI>(a, s);
    case 4: return run_sum_ks<4, EPI>(a, s);
    case 5: return run_sum_ks<5, EPI>(a, s);
    case 6: return run_sum_ks<6, EPI>(a, s);
    case 7: return run_sum_ks<7, EPI>(a, s);
    case 8: return run_sum_ks<8, EPI>(a, s);
  }
  return hipErrorInvalidValue;
}

template <int EPI>
hipError_t run_dma(GemmArgs a, hipStream_t s, int* np, const GemmTiles* given) {
  if (!a.ncg) {  // planes: this product's activations in fragment order first
    a.ncg = (a.R + 7) / 8;
    const int64_t frags = (int64_t)(a.K >> 5) * a.ncg;
    if (!a.xfrag || (size_t)frags * 512 > a.xfrag_elems) return hipErrorInvalidValue;
    hipLaunchKernelGGL(xfrag_kernel, dim3((unsigned)((frags + 3) / 4)), dim3(256), 0, s, a.X, a.xfrag, a.R, a.K, a.ncg);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    a.X = a.xfrag;
  }
  const Plan p = given ? plan_of(a, *given) : plan_for(a, EPI);
  hipError_t e = hipErrorInvalidValue;
  if (p.tall) switch (p.A) {
    case 5: e = run_tall<5, EPI>(a, p, s); break;
    case 6: e = run_tall<6, EPI>(a, p, s); break;
    case 7: e = run_tall<7, EPI>(a, p, s); break;
    case 8: e = run_tall<8, EPI>(a, p, s); break;
  }
  else switch (p.A) {
    case 4: e = run_rows<4, EPI>(a, p, s); break;
    case 5: e = run_rows<5, EPI>(a, p, s); break;
    case 6: e = run_rows<6, EPI>(a, p, s); break;
    case 7: e = run_rows<7, EPI>(a, p, s); break;
    case 8: e = run_rows<8, EPI>(a, p, s); break;
  }
  if (e != hipSuccess) return e;
  if (p.KS > 1) e = run_sum<EPI>(a, p.KS, s);
  if (np) *np = p.KS > 1 ? row_pieces(a.N) : a.N >> 4;
  return e;
}

}  // namespace

size_t gemm_dma_xfrag_elems(int R, int K) { return (size_t)(K >> 5) * ((R + 7) / 8) * 512; }

// floats of workspace the ranges of a cut reduction may take: at most one workgroup per compute unit, 256 rows x 16 strips each
size_t gemm_dma_split_floats() { return (size_t)device_cus() * 256 * 256; }

bool gemm_dma_wide(int N) { return ((N >> 4) + 7) / 8 * 2 >= device_cus(); }

GemmTiles gemm_dma_tiles(const GemmArgs& a, int epi) {
  const Plan p = plan_for(a, epi);
  return GemmTiles{p.A, p.B, p.tall, p.KS, 0};
}

hipError_t launch_gemm_bf16_dma(const GemmArgs& a, int epi, hipStream_t s, int* np, const GemmTiles* t) {
  if (t) {  // what plan_for and launch_gemm_bf16 see to for planned tiles
    if (a.R <= ACT_COMPACT_ROWS || (a.N & 15) || (a.K & 31) || (epi == EPI_STORE && (a.ldy & 3))) return hipErrorInvalidValue;
    if (t->ranges < 1 || (t->ranges > 1 && !(can_cut(a, epi) && cut_fits(a, t->ranges)))) return hipErrorInvalidValue;
    if (t->tall < 0 || t->tall > 1 || t->strips < 4) return hipErrorInvalidValue;
    if (t->tall ? t->strips < 5 || t->strips > 8 || t->row_groups < 3 || t->row_groups > 4
                : t->strips > 8 || t->row_groups < 0 || t->row_groups > (t->strips == 4 ? 1 : 4))
      return hipErrorInvalidValue;
  }
  switch (epi) {
    case EPI_STORE: return run_dma<EPI_STORE>(a, s, np, t);
    case EPI_RESID: return run_dma<EPI_RESID>(a, s, np, t);
    case EPI_SWIGLU: return run_dma<EPI_SWIGLU>(a, s, np, t);
    case EPI_QKV: return run_dma<EPI_QKV>(a, s, np, t);
  }
  return hipErrorInvalidValue;
}

}  // namespace mtad

// For the tests (and to time plans against each other): the many-row product with the epilogue and the tiles named, tiles[4] =
// {strips per wave, row groups of 64 (0: one of 32), groups side by side, ranges}, or, with tiles[0] = 0, the planned tiles
// written there.  args: a GemmArgs of `bytes` bytes.  run 0: no launch; above 1: on a device taken to have that many bytes of LDS
// per compute unit.  0, or -1 (sizes differ, or tiles that do not exist or fit) or -4.
extern "C" int mtad_test_gemm_tiles(const void* args, size_t bytes, int epi, int* tiles, int run, void* stream) {
  using namespace mtad;
  if (!args || !tiles || bytes != sizeof(GemmArgs)) return -1;
  const GemmArgs& a = *(const GemmArgs*)args;
  GemmTiles t{tiles[0], tiles[1], tiles[2], tiles[3], run > 1 ? run : 0};
  if (!t.strips) t = gemm_dma_tiles(a, epi);
  tiles[0] = t.strips; tiles[1] = t.row_groups; tiles[2] = t.tall; tiles[3] = t.ranges;
  if (!run) return 0;
  const hipError_t e = launch_gemm_bf16_dma(a, epi, (hipStream_t)stream, nullptr, &t);
  return e == hipSuccess ? 0 : e == hipErrorInvalidValue ? -1 : -4;
}
