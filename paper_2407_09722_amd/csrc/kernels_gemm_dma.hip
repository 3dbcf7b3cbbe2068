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
//     matrix instructions.  An interval is one k tile.  k tile j lies in ring slot j % D; it is read in interval j, its slot is refilled with k tile j + D in interval j + 1 (after the barrier
//     that ends the reads), and every wave waits for its own share of k tile j + 1 before the barrier that ends interval j.
//   * an activation fragment holds 8 rows, hi and lo in alternate 128-byte pieces; a B operand takes every other piece of two
//     fragments (shifting the second one by 128 bytes, so that an LDS beat touches other banks, measured the same).
// Measured (us per launch, the kernel before this one -> this one): 27648 x 5120 at 164 rows 122 -> 104 and at 256 rows 193 -> 133
// (1.09 PFLOP/s, hi and lo counted), 15360 x 5120 at 164 rows 90 -> 66, 5120 x 5120 51 -> 30, 5120 x 13824 96 -> 61, 22016 x 4096
// at 64 rows 48 -> 43.  At 256 rows of the first shape the matrix instructions alone take 88 us, the activations' way to LDS 61 and
// the weights' 60 (24 of each are launch, epilogue and barriers), all together 133: a compute unit's loads return in the order
// they were made, so activations that lie in L2 wait behind weights that come from HBM, and the two do not overlap.
#include "common.h"
#include "gemm.h"
#include "gemm_device.h"

#include <atomic>

namespace mtad {

namespace {

constexpr int NW = 8;                    // waves per workgroup: two groups of four
constexpr int LDS_MOST = 160 * 1024 - 1536;  // of a compute unit, less the static arrays
constexpr int PAIR = 2048;  // bytes of two activation fragments (16 rows)

template <int A, int B>
struct DmaShape {
  static constexpr int ROWS = 64 * B;                // rows per workgroup
  static constexpr int A0 = (A + 1) / 2;             // strips group 0 finishes
  static constexpr int FRAGS = A + 8 * B;            // KiB that one k tile brings: A weight tiles, then 8 B activation fragments
  static constexpr int LPW = (FRAGS + NW - 1) / NW;  // of them per wave
  static constexpr int SLOT = A * 1024 + 4 * B * PAIR;
  static constexpr int D0 = LDS_MOST / SLOT;
  static constexpr int D = D0 > 16 ? 16 : D0;         // ring slots
  static_assert(D >= 3, "one slot read, one arriving, one being requested");
  static constexpr int RED = 4 * 64 * 16 * B * A;    // bytes the groups exchange
  static constexpr int LDS = D * SLOT > RED ? D * SLOT : RED;
  static_assert((D - 2) * LPW <= 63, "wait counter");
  static_assert(LDS + ROWS * 4 <= 160 * 1024, "a compute unit's LDS");
};

// s_waitcnt operand (gfx9 encoding): at most n vector memory operations outstanding, no LDS operation
constexpr int wait_vm_lds(int n) { return (n & 15) | ((n >> 4) << 14) | 0x0070; }

typedef const __attribute__((address_space(1))) uint32_t* GlobalWords;
typedef __attribute__((address_space(3))) uint32_t* LdsWords;

template <int A, int B, int EPI>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(2, 2))) void gemm_bf16_dma_kernel(GemmArgs a, int tiles_n, int tiles_m, int KS) {
  using Sh = DmaShape<A, B>;
  constexpr int LPW = Sh::LPW, D = Sh::D, SLOT = Sh::SLOT;
  extern __shared__ __attribute__((aligned(16))) unsigned char lds_dma[];
  __shared__ float inv_s[Sh::ROWS];

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wr = wave & 3, grp = wave >> 2;
  const int c = lane & 15, kg = lane >> 4;
  const int KT_all = a.K >> 5, NT = a.N >> 4;
  // workgroups go to the 8 XCDs in turn: give each XCD a contiguous range of tiles, and within it blocks of up to four row tiles
  // by a few feature tiles, so that its L2 serves a weight tile to four workgroups and an activation fragment to several
  const int total = (int)gridDim.x, id = (int)blockIdx.x, xcd = id & 7;
  int l = xcd * (total >> 3) + min(xcd, total & 7) + (id >> 3);
  const int tiles = tiles_n * tiles_m, ks = l / tiles;
  l -= ks * tiles;
  const int per_group = 4 * tiles_n, mg = l / per_group, lg = l - mg * per_group;
  const int gm = min(4, tiles_m - mg * 4);
  const int tm = mg * 4 + lg % gm, tn = lg / gm;
  const int nt0 = tn * A, row0 = tm * Sh::ROWS;
  const int per = (KT_all + KS - 1) / KS, k_lo = ks * per;
  const int n_kt = min(KT_all, k_lo + per) - k_lo;  // the launcher leaves no range empty

  // What this wave requests per k tile: fragment f = i * 8 + wave is weight tile f, or activation fragment f - A; those past
  // the last one read it again, to the same place with the same contents.  (Weights on waves of their own, requested much
  // earlier than the activations, were no faster: a compute unit's loads return in the order of their requests, so the
  // activations behind them wait for HBM all the same, and the ring holds fewer of them.)
  const char* src[LPW];
  size_t step[LPW];
  unsigned dst[LPW];
  const int cg0 = row0 >> 3, cg_last = a.ncg - 1;
#pragma unroll
  for (int i = 0; i < LPW; ++i) {
    const int f = min(i * NW + wave, Sh::FRAGS - 1);
    if (f < A) {
      src[i] = (const char*)a.W + (((size_t)min(nt0 + f, NT - 1) * KT_all + k_lo) << 10);
      step[i] = 1024;
      dst[i] = (unsigned)f * 1024u;
    } else {
      const int x = f - A;
      src[i] = (const char*)a.X + (((size_t)k_lo * a.ncg + min(cg0 + x, cg_last)) << 10);
      step[i] = (size_t)a.ncg << 10;
      dst[i] = (unsigned)(A * 1024 + x * 1024);
    }
  }
  int s_in = 0;  // ring slot of the next request, in bytes
  auto request = [&]() {
#pragma unroll
    for (int i = 0; i < LPW; ++i) {
      __builtin_amdgcn_global_load_lds((GlobalWords)(src[i] + (unsigned)lane * 16u), (LdsWords)(lds_dma + s_in + dst[i]), 16, 0, 0);
      src[i] += step[i];
    }
    s_in = s_in + SLOT == D * SLOT ? 0 : s_in + SLOT;
  };
  constexpr int ahead = D - 1;
  for (int j = 0; j < ahead && j < n_kt; ++j) request();
  {
    GemmArgs ar = a;
    ar.row0 = row0;
    gemm_row_factors<false, 8>(ar, inv_s, min(Sh::ROWS, a.R - row0), wave, lane, NW);
  }

  floatx4 acc[A][B];
#pragma unroll
  for (int si = 0; si < A; ++si)
#pragma unroll
    for (int j = 0; j < B; ++j) acc[si][j] = floatx4{0.f, 0.f, 0.f, 0.f};
  // lane (kg, row) of a B operand: fragment row / 8 of the pair, piece (kg, plane), row % 8
  const unsigned w_off = (unsigned)lane * 16u;
  const unsigned x_off = (unsigned)(A * 1024 + wr * PAIR + (c >> 3) * 1024 + (kg * 16 + (c & 7)) * 16);
  Frag fw[A], fx[B][2];
  int s_out = grp * SLOT;  // ring slot of this group's next k tile
  auto fetch = [&]() {
    const unsigned char *const wp = lds_dma + s_out + w_off, *const xp = lds_dma + s_out + x_off;
#pragma unroll
    for (int si = 0; si < A; ++si) fw[si].n = *(const uintx4*)(wp + si * 1024);
#pragma unroll
    for (int j = 0; j < B; ++j) {
      fx[j][0].n = *(const uintx4*)(xp + j * (4 * PAIR));
      fx[j][1].n = *(const uintx4*)(xp + j * (4 * PAIR) + 128);
    }
    s_out += 2 * SLOT;
    if (s_out >= D * SLOT) s_out -= D * SLOT;
  };
  // An interval ends: this wave's requests for the next k tile have arrived (all but its requests for later ones, or all
  // of them when it has no more to make), its fragment reads are done, then the barrier.  The fences keep the compiler
  // from moving memory operations across (the barrier alone does not).
  auto interval_end = [&](bool steady) {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
    if (steady) __builtin_amdgcn_s_waitcnt(wait_vm_lds((D - 2) * LPW));
    else __builtin_amdgcn_s_waitcnt(wait_vm_lds(0));
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };

  interval_end(n_kt >= ahead);  // k tile 0 is there (and the row factors)
  int i = 0;  // interval: k tile i + ahead is requested in it
  if (grp == 1) {
    const bool more = i + ahead < n_kt;
    if (more) request();
    interval_end(more);
    ++i;
  }
  const int trips = (n_kt + 1) >> 1;
#pragma unroll 1
  for (int t = 0; t < trips; ++t) {
    // memory interval: fragments of this group's k tile
    {
      const bool more = i + ahead < n_kt;
      fetch();
      if (more) request();
      interval_end(more);
      ++i;
    }
    // compute interval
    {
      const bool more = i + ahead < n_kt;
      if (more) request();
      __builtin_amdgcn_sched_barrier(0);
      if (grp == 0 || 2 * t + 1 < n_kt) {
#pragma unroll
        for (int j = 0; j < B; ++j)
#pragma unroll
          for (int p = 0; p < 2; ++p)
#pragma unroll
            for (int si = 0; si < A; ++si) acc[si][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fw[si].v, fx[j][p].v, acc[si][j], 0, 0, 0);
      }
      interval_end(more);
      ++i;
    }
  }
  if (grp == 0) interval_end(false);

  // the groups' sums meet in LDS: group 0 finishes strips 0 .. A0 - 1, group 1 the others
  constexpr int A0 = Sh::A0;
  floatx4* const red = reinterpret_cast<floatx4*>(lds_dma);  // [4 waves][A][B][64]
#pragma unroll
  for (int si = 0; si < A; ++si)
    if ((si < A0) == (grp == 1)) {
#pragma unroll
      for (int j = 0; j < B; ++j) red[((wr * A + si) * B + j) * 64 + lane] = acc[si][j];
    }
  __syncthreads();
  const int rows_here = min(Sh::ROWS, a.R - row0);
#pragma unroll
  for (int si = 0; si < A; ++si)
    if ((si < A0) == (grp == 0) && nt0 + si < NT) {
      const int nt = nt0 + si;
      floatx4 s[B];
#pragma unroll
      for (int j = 0; j < B; ++j) {
        const floatx4 o = red[((wr * A + si) * B + j) * 64 + lane];
        // even k tiles first, whichever group adds
#pragma unroll
        for (int e = 0; e < 4; ++e) s[j][e] = acc[si][j][e] + o[e];
      }
      if (KS > 1) {  // the launch after this one adds the ranges: part[range][row][feature]
#pragma unroll
        for (int j = 0; j < B; ++j) {
          const int mrel = (j * 4 + wr) * 16 + c;
          if (mrel < rows_here) *(floatx4*)(a.part + ((size_t)ks * a.R + row0 + mrel) * a.N + nt * 16 + kg * 4) = s[j];
        }
      } else {
        float4 ph[B], pg = float4{0.f, 0.f, 0.f, 0.f};
        if constexpr (EPI == EPI_RESID) {  // the residual values of all row groups first: one latency, not B
          pg = *(const float4*)(a.g_next + nt * 16 + kg * 4);
#pragma unroll
          for (int j = 0; j < B; ++j) {
            const int mrel = min((j * 4 + wr) * 16 + c, rows_here - 1);
            ph[j] = *(const float4*)(a.h + (int64_t)(row0 + mrel) * a.N + nt * 16 + kg * 4);
          }
        }
#pragma unroll
        for (int j = 0; j < B; ++j) {
          const int mrel = (j * 4 + wr) * 16 + c;
          const bool live = mrel < rows_here;
          const float inv = (a.ssq && live) ? inv_s[mrel] : 1.0f;
          gemm_epilogue<EPI, false, EPI == EPI_RESID>(a, nt, s[j], row0 + mrel, live, inv, kg, ph[j], pg);
        }
      }
    }
}

// After a product whose reduction dimension was cut into KS ranges: one workgroup per row adds the ranges in order.
//   RESID  the residual epilogue over the whole row: h += sum, the next norm's input h * gain as hi / lo terms, and the row's
//          sum of squares as ONE value, so that the products that read it have nothing left to reduce
//   STORE  the row of Y
constexpr int RT = 1024;  // threads
template <int KS, int EPI>
__global__ __launch_bounds__(RT) void gemm_rows_kernel(GemmArgs a) {
  __shared__ float sh[RT / 64];
  const int m = blockIdx.x, N = a.N;
  const size_t range = (size_t)a.R * N;
  float q = 0.f;
  for (int n = (int)threadIdx.x * 4; n < N; n += RT * 4) {
    const float* const p = a.part + (size_t)m * N + n;
    float4 t[KS];
#pragma unroll
    for (int k = 0; k < KS; ++k) t[k] = *(const float4*)(p + k * range);
    float4 s = t[0];
#pragma unroll
    for (int k = 1; k < KS; ++k) { s.x += t[k].x; s.y += t[k].y; s.z += t[k].z; s.w += t[k].w; }
    if constexpr (EPI == EPI_STORE) {
      float4* const y = (float4*)(a.Y + (int64_t)m * a.ldy + n);
      if (a.accumulate) {
        const float4 o = *y;
        s.x += o.x; s.y += o.y; s.z += o.z; s.w += o.w;
      }
      *y = s;
    } else {
      float4* const hp = (float4*)(a.h + (int64_t)m * N + n);
      const float4 o = *hp, gn = *(const float4*)(a.g_next + n);
      s.x += o.x; s.y += o.y; s.z += o.z; s.w += o.w;
      *hp = s;
      ushort4 hi, lo;
      split_bf16(s.x * gn.x, hi.x, lo.x);
      split_bf16(s.y * gn.y, hi.y, lo.y);
      split_bf16(s.z * gn.z, hi.z, lo.z);
      split_bf16(s.w * gn.w, hi.w, lo.w);
      *(ushort4*)(a.planes_out + act_offset(a.ncg, a.R, N, 0, m, n)) = hi;
      *(ushort4*)(a.planes_out + act_offset(a.ncg, a.R, N, 1, m, n)) = lo;
      q += s.x * s.x + s.y * s.y + s.z * s.z + s.w * s.w;
    }
  }
  if constexpr (EPI == EPI_RESID) {
    for (int off = 32; off > 0; off >>= 1) q += __shfl_xor(q, off, 64);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = q;
    __syncthreads();
    if (threadIdx.x == 0) {
      for (int w = 1; w < RT / 64; ++w) q += sh[w];
      a.ssq_out[m] = q;
    }
  }
}

// Sums of squares of a pass of many rows, [R][NP] -> [R]: every workgroup of the products that read them would otherwise reduce
// its 256 rows again.
__global__ __launch_bounds__(256) void ssq_rows_kernel(const float* __restrict__ in, float* __restrict__ out, int R, int NP) {
  const int m = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (m >= R) return;
  float s = 0.f;
  for (int p = lane; p < NP; p += 64) s += in[(int64_t)m * NP + p];
  for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
  if (lane == 0) out[m] = s;
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

struct Plan {
  int A, B, KS, tiles_n, tiles_m;
};
constexpr int KS_MAX = 8;

// Rows per workgroup: row tiles of at most 256 rows, as equal as steps of 64 allow.  Strips per workgroup (4 to 8) and ranges of
// the reduction dimension: the cheapest by a count of clocks per compute unit.  An interval (one k tile) lasts as long as its
// matrix instructions, its LDS traffic or its weights from HBM (about 10 bytes per clock and compute unit), plus the barrier.
// A cut costs its partial sums' way through memory and a launch.
Plan plan_for(const GemmArgs& a, int epi) {
  Plan best{};
  const int NT = a.N >> 4, KT = a.K >> 5, cus = device_cus();
  const int tm = (a.R + 255) / 256, B = ((a.R + tm - 1) / tm + 63) / 64;
  double best_cost = 0;
  for (int A = 8; A >= 4; --A) {
    const int tn = (NT + A - 1) / A;
    const int mfma = 32 * A * B, lds = 32 * (A + 2 * B) + 8 * (A + 8 * B), hbm = 98 * A;
    const int interval = (mfma > lds ? (mfma > hbm ? mfma : hbm) : (lds > hbm ? lds : hbm)) + 100;
    for (int KS = 1; KS <= KS_MAX; ++KS) {
      const int total = tn * tm * KS;
      if (KS > 1) {
        if (!a.part || (epi != EPI_RESID && !(epi == EPI_STORE && !a.lse_part && !a.ssq))) break;
        if (total > cus || KT < 16 * KS || (size_t)KS * a.R * a.N > a.part_floats) break;
        if (((KT + KS - 1) / KS) * (KS - 1) >= KT) continue;  // a range would be empty
      }
      const int rounds = (total + cus - 1) / cus;
      double cost = (double)rounds * (((KT + KS - 1) / KS) * (double)interval + 8000);
      if (KS > 1) cost += 6000 + (double)(2 * KS) * a.R * a.N * 4 / 2000;
      if (best.A == 0 || cost < best_cost) {
        best_cost = cost;
        best = Plan{A, B, KS, tn, tm};
      }
    }
  }
  return best;
}

template <int A, int B, int EPI>
hipError_t run_shape(const GemmArgs& a, const Plan& p, hipStream_t s) {
  using Sh = DmaShape<A, B>;
  auto kern = gemm_bf16_dma_kernel<A, B, EPI>;
  // more than 64 KiB of dynamic LDS needs the attribute; a success is remembered, a failure is reported and tried again
  static std::atomic<bool> attr_set{false};
  if (!attr_set.load(std::memory_order_acquire)) {
    const hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, Sh::LDS);
    if (e != hipSuccess) return e;
    attr_set.store(true, std::memory_order_release);
  }
  hipLaunchKernelGGL(kern, dim3((unsigned)(p.tiles_n * p.tiles_m * p.KS)), dim3(NW * 64), Sh::LDS, s, a, p.tiles_n, p.tiles_m, p.KS);
  return hipGetLastError();
}

template <int A, int EPI>
hipError_t run_rows(const GemmArgs& a, const Plan& p, hipStream_t s) {
  switch (p.B) {
    case 1: return run_shape<A, 1, EPI>(a, p, s);
    case 2: return run_shape<A, 2, EPI>(a, p, s);
    case 3: return run_shape<A, 3, EPI>(a, p, s);
    case 4: return run_shape<A, 4, EPI>(a, p, s);
  }
  return hipErrorInvalidValue;
}

template <int EPI>
hipError_t run_sum(const GemmArgs& a, int KS, hipStream_t s) {
  const dim3 grid((unsigned)a.R), block(RT);
  switch (KS) {
    case 2: hipLaunchKernelGGL((gemm_rows_kernel<2, EPI>), grid, block, 0, s, a); break;
    case 3: hipLaunchKernelGGL((gemm_rows_kernel<3, EPI>), grid, block, 0, s, a); break;
    case 4: hipLaunchKernelGGL((gemm_rows_kernel<4, EPI>), grid, block, 0, s, a); break;
    case 5: hipLaunchKernelGGL((gemm_rows_kernel<5, EPI>), grid, block, 0, s, a); break;
    case 6: hipLaunchKernelGGL((gemm_rows_kernel<6, EPI>), grid, block, 0, s, a); break;
    case 7: hipLaunchKernelGGL((gemm_rows_kernel<7, EPI>), grid, block, 0, s, a); break;
    case 8: hipLaunchKernelGGL((gemm_rows_kernel<8, EPI>), grid, block, 0, s, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <int EPI>
hipError_t run_dma(GemmArgs a, hipStream_t s, int* np) {
  if (!a.ncg) {  // planes: this product's activations in fragment order first
    a.ncg = (a.R + 7) / 8;
    const int64_t frags = (int64_t)(a.K >> 5) * a.ncg;
    if (!a.xfrag || (size_t)frags * 512 > a.xfrag_elems) return hipErrorInvalidValue;
    hipLaunchKernelGGL(xfrag_kernel, dim3((unsigned)((frags + 3) / 4)), dim3(256), 0, s, a.X, a.xfrag, a.R, a.K, a.ncg);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    a.X = a.xfrag;
  }
  const Plan p = plan_for(a, EPI);
  hipError_t e = hipErrorInvalidValue;
  switch (p.A) {
    case 4: e = run_rows<4, EPI>(a, p, s); break;
    case 5: e = run_rows<5, EPI>(a, p, s); break;
    case 6: e = run_rows<6, EPI>(a, p, s); break;
    case 7: e = run_rows<7, EPI>(a, p, s); break;
    case 8: e = run_rows<8, EPI>(a, p, s); break;
  }
  if (e != hipSuccess) return e;
  if constexpr (EPI == EPI_RESID || EPI == EPI_STORE) {
    if (p.KS > 1) e = run_sum<EPI>(a, p.KS, s);
  }
  if (np) *np = p.KS > 1 ? 1 : a.N >> 4;
  return e;
}

}  // namespace

size_t gemm_dma_xfrag_elems(int R, int K) { return (size_t)(K >> 5) * ((R + 7) / 8) * 512; }

// floats of workspace the ranges of a cut reduction may take: at most one workgroup per compute unit, 256 rows x 8 strips each
size_t gemm_dma_split_floats() { return (size_t)device_cus() * 256 * 128; }

hipError_t launch_ssq_rows(const float* in, float* out, int R, int NP, hipStream_t s) {
  hipLaunchKernelGGL(ssq_rows_kernel, dim3((unsigned)((R + 3) / 4)), dim3(256), 0, s, in, out, R, NP);
  return hipGetLastError();
}

bool gemm_dma_wide(int N) { return ((N >> 4) + 7) / 8 * 2 >= device_cus(); }

hipError_t launch_gemm_bf16_dma(const GemmArgs& a, int epi, hipStream_t s, int* np) {
  switch (epi) {
    case EPI_STORE: return run_dma<EPI_STORE>(a, s, np);
    case EPI_RESID: return run_dma<EPI_RESID>(a, s, np);
    case EPI_SWIGLU: return run_dma<EPI_SWIGLU>(a, s, np);
    case EPI_QKV: return run_dma<EPI_QKV>(a, s, np);
  }
  return hipErrorInvalidValue;
}

}  // namespace mtad
