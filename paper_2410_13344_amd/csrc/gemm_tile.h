// Whole-K GEMMs with fused epilogues for launches of more than 64 rows (bf16 mode): the QKV projection with RoPE and the KV
// write, and the gate/up projection with SwiGLU.  The O and down projections, with few columns, run on the same tiles over ranges of
// K and leave fp32 planes.
//
// A workgroup of 8 waves per compute unit owns a row block (at most 128 rows) and a few 16-column slabs over the full K, so
// there are no partial planes: the epilogue works on finished sums and no consumer kernel follows.  Row blocks and column
// groups are formed on the device from the step's row count (the host knows a bound only): the fewest row blocks of at most
// 128 rows, two above 64 rows; the slabs, in pairs whose columns an epilogue needs together, are dealt evenly to the
// workgroups of a row block; what does not fit the accumulators (12 pairs) goes in rounds.
//
// Both operands go global -> LDS by direct loads in MFMA fragment order, several stages deep, and are shared: the waves
// stand 2 x 4 (half of the row tiles by every fourth pair) or 4 x 2, whichever reads less from LDS.  The fragments of the next
// k-step are read from LDS while this one is multiplied, across the barrier between stages too (a stage has landed for
// everyone one barrier before its turn).  What that is worth, gate/up of the 7B shape (K = 4096, N = 22016), bare kernel: 323
// rows 149 us with the reads in front of the products, 116 with them a k-step ahead; 121 rows 71 and 57; 1024 rows 330 and
// 306.  A stage is 40 pieces of 1 KB at most; small tiles take two k-steps per stage (121 rows 57 us, with one 71).  Bounds: at
// 121 rows what the L2s and HBM deliver into a compute unit (A and the slabs come in at 13-15 TB/s over the chip, 53 us of the
// 57); at 1024 rows the matrix cores at the clock the load leaves them (250-265 us without any loads).  In between neither alone:
// at 323 rows gate/up brings in 1.03 GB in 114-116 us (9 TB/s) with the matrix cores busy 42 % of the time, QKV 0.78 GB in 82 us
// with 33 %; loads and products add up more than they overlap.
//
// The matrix cores round a running sum with every product, so the error of a sum grows with its length, and a
// cached element whose sum is off by little moves by a whole step of bf16 now and then.  So every 8 k-steps the sums move
// over to a second set of accumulators.  A wave's tile of 3 or 4 x 3 has registers for a second set only where its slab fragments
// are refilled in place and the addresses of its loads are scalar (kWide): gate/up, and down where its input lies in fragments,
// whose sums move over every 32 k-steps there.  The others have no such tiles: QKV takes fewer pairs per round, row-major A more
// k ranges.  (Without a second set sums of 3670 to 6912 columns of down were off by 2.9e-7 to 5.3e-7 of the result where all
// products are positive, the others by 1e-7.)
//
// The products are W A^T: a lane then holds four consecutive columns of one row, which go out as one store per plane.
#pragma once
#include <type_traits>

#include "step_kernels.h"

namespace cerb {

namespace {   // (a copy per source that includes this, each with kernels of its own)

constexpr int kTileLds = 160 * 1024;
constexpr int kMaxPairs = 12;   // of a round: three per wave of 2 x 4
constexpr int kSumSteps = 8;    // k-steps of a sum
constexpr int kSumStepsWide = 32;   // ... on a tile of more than
constexpr int kMaxTwo = 8;      // row tiles x pairs of a wave, which leave room for two sets of slab fragments

__device__ __forceinline__ void tile_dma16(const char* p, unsigned lds_addr) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds_addr), "v"(p) : "memory", "m0");
}
// The same from a wave-uniform address and a lane's offset.  The wait states in front: a scalar register written by the vector
// unit (v_readfirstlane, or v_readlane where the compiler reloads a spilled one) may be read as an address five wait states later
// at the earliest, and the compiler does not see to that inside inline assembly.
__device__ __forceinline__ void tile_dma16(const char* base, unsigned off, unsigned lds_addr) {
  asm volatile("s_nop 4\n\ts_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds_addr), "v"(off), "s"(base) : "memory", "m0");
}
__device__ __forceinline__ const char* tile_uniform(const char* p) {
  const unsigned long v = reinterpret_cast<unsigned long>(p);
  const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)v), hi = __builtin_amdgcn_readfirstlane((unsigned)(v >> 32));
  return reinterpret_cast<const char*>(((unsigned long)hi << 32) | lo);
}

// Row tiles [m0/16, m0/16 + nmt) by pairs [p0, p0 + np) of the launch
// over k-steps [ks0, ks0 + nks), both multiples of 8; split: the number of the k range
struct TileJob { int m0, m1, nmt, p0, np, rounds, perr, ks0, nks, split; };

// KC k-steps per stage, CW pieces of 1 KB per wave and stage, WR x WC waves
template <int KC, int CW, int WR, typename Epi>
__device__ __forceinline__ void tile_run(const TileGemmArgs& a, const TileJob& J, const Epi& epi, u32x4_t* lds) {
  constexpr int WC = 8 / WR;
  constexpr unsigned SB = CW * 8 * 1024;
  constexpr int D = kTileLds / (int)SB;                        // stages in LDS
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int nst = J.nks / KC;
  // row group and pair group of the wave; waves w and w + 4 share a SIMD: what the larger groups take is spread over the SIMDs
  const int wl = wave & 3, wh = wave >> 2;
  const int rg = WR == 2 ? wh : wh ? 3 - wl : wl, cg = WR == 4 ? wh : wh ? 3 - wl : wl;
  const int rt = (J.nmt + WR - 1 - rg) / WR, t0 = rg * (J.nmt / WR) + min(rg, J.nmt % WR);
  const int P1 = 2 * J.nmt + 2 * J.perr;                       // pieces per k-step: A (row tile, plane), then W (pair, slab)
  const unsigned ldsb = (unsigned)(unsigned long)((__attribute__((address_space(3))) const unsigned char*)lds);

  // ---- pieces q * 8 + wave of a stage (past the last one: that one once more, into a slot nobody reads)
  constexpr bool SADDR = Epi::kWide;                           // src: the wave's address; else the lane's
  const char* src[CW];
  unsigned step[CW];
  auto bases = [&](int rd) {
    int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    asm volatile("" : "+v"(lane));                             // (nothing of this is kept in registers from round to round)
    asm volatile("" : "+s"(wave));
#pragma unroll
    for (int q = 0; q < CW; ++q) {
      const int p = min(q * 8 + wave, KC * P1 - 1), kc = KC == 2 && p >= P1 ? 1 : 0, r = p - kc * P1;
      if (r < 2 * J.nmt) {
        if (Epi::kRows) {   // 64 bytes of each of 16 rows
          src[q] = reinterpret_cast<const char*>(a.A) + ((r & 1) * a.lo_off + (size_t)min(J.m0 + (r >> 1) * 16 + (lane & 15), J.m1 - 1) * a.lda + (J.ks0 + kc) * 32 + (lane >> 4) * 8) * 2;
          step[q] = KC * 64;
          continue;
        } else {
          src[q] = reinterpret_cast<const char*>(a.A) + ((size_t)((size_t)(J.m0 / 16 + (r >> 1)) * a.ksteps + J.ks0 + kc) * 2 + (r & 1)) * 1024;
          step[q] = KC * 2048;
        }
      } else {
        const int pos = r - 2 * J.nmt, pair = min(J.p0 + rd * J.perr + (pos >> 1), J.p0 + J.np - 1);
        src[q] = reinterpret_cast<const char*>(a.W) + ((size_t)epi.slab(pair, pos & 1) * a.ksteps + J.ks0 + kc) * 1024;
        step[q] = KC * 1024;
      }
      if constexpr (SADDR) {
        src[q] = tile_uniform(src[q]);
        step[q] = __builtin_amdgcn_readfirstlane(step[q]);
      } else {
        src[q] += lane * 16;
      }
    }
  };
  bases(0);
  int ist = 0, ird = 0, ibuf = 0, left = nst * J.rounds;       // the stage to be issued; issues past the last repeat it
  auto issue = [&](auto wraps) {                               // wraps: the stage may be a round's last one
    const unsigned l0 = __builtin_amdgcn_readfirstlane(ldsb + ibuf * SB + wave * 1024);
#pragma unroll
    for (int q = 0; q < CW; ++q) {
      if constexpr (SADDR) {
        tile_dma16(src[q], lane * 16, l0 + q * 8192);
      } else {
        tile_dma16(src[q], l0 + q * 8192);
      }
    }
    ibuf = ibuf + 1 == D ? 0 : ibuf + 1;
    if (left > 1) {
      --left;
      ++ist;
      if (decltype(wraps)::value && ist == nst) {
        ist = 0;
        bases(++ird);
      } else {
#pragma unroll
        for (int q = 0; q < CW; ++q) src[q] += step[q];
      }
    }
  };
#pragma unroll 1
  for (int i = 0; i < D - 1; ++i) issue(std::true_type{});

  int buf = 0;
  // Top of stage n: this wave's pieces of stage n + 1 have landed, then everyone's; and everyone has multiplied stage n - 1,
  // whose buffer takes stage n + D - 1 (no lgkmcnt: a read that still runs here is one of stage n's first fragments).
  auto top = [&](auto wraps) {
    asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"((D - 3) * CW) : "memory");
    issue(wraps);
  };
  auto multiply = [&](auto rtc, auto nqc, int rd) {
    constexpr int RT = decltype(rtc)::value, NQ = decltype(nqc)::value, NW = 2 * NQ;
    const u32x4_t* la = lds + lane + t0 * 128;
    const u32x4_t* lw = lds + lane + (2 * J.nmt + cg * 2) * 64;
    constexpr bool WIDE = RT * NQ > kMaxTwo;                   // slab fragments are refilled in place
    constexpr int SUM = (WIDE ? kSumStepsWide : kSumSteps) / KC;
    f32x4_t acc[RT][NW], tot[RT][NW];
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
      for (int j = 0; j < NW; ++j) acc[i][j] = tot[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    int sum_left = SUM;
    u32x4_t w[WIDE ? 1 : 2][NW], fa[2][2];                     // this k-step's slabs and the next one's; a row tile and the next
    auto rdw = [&](u32x4_t (&d)[NW], const u32x4_t* s, int j) { d[j] = s[(j >> 1) * (WC * 128) + (j & 1) * 64]; };
    const unsigned p1 = P1 * 64;
    for (int st = 0; st < nst; st += (KC == 1 ? 2 : 1)) {      // two k-steps per trip
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        // (a round's last stage is issued at the top of stage n with n + D a multiple of nst, which is even for one k-step a stage)
        if (KC == 2 && h == 0) top(std::true_type{});
        if (KC == 1 && h == D % 2) top(std::true_type{});
        if (KC == 1 && h != D % 2) top(std::false_type{});
        const int nbuf = buf + 1 == D ? 0 : buf + 1;
        const unsigned cb = buf * (SB / 16) + (KC == 2 && h == 1 ? p1 : 0);
        const unsigned nb = KC == 2 && h == 0 ? buf * (SB / 16) + p1 : nbuf * (SB / 16);
        const u32x4_t *ca = la + cb, *cw = lw + cb, *na = la + nb, *nw = lw + nb;
        if (KC == 1 || h == 1) buf = nbuf;
        if (h == 0 && st == 0) {
#pragma unroll
          for (int j = 0; j < NW; ++j) rdw(w[0], cw, j);
          fa[0][0] = ca[0];
          fa[0][1] = ca[64];
        }
#pragma unroll
        for (int i = 0; i < RT; ++i) {
          const int cur = (h * RT + i) & 1;
          const u32x4_t* nx = i + 1 < RT ? ca + (i + 1) * 128 : na;
          fa[cur ^ 1][0] = nx[0];
          fa[cur ^ 1][1] = nx[64];
          if constexpr (!WIDE) {
#pragma unroll
            for (int j = i * NW / RT; j < (i + 1) * NW / RT; ++j) rdw(w[h ^ 1], nw, j);
          }
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int j = 0; j < NW; ++j) {
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, w[WIDE ? 0 : h][j]), __builtin_bit_cast(bf16x8_t, fa[cur][0]), acc[i][j], 0, 0, 0);
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, w[WIDE ? 0 : h][j]), __builtin_bit_cast(bf16x8_t, fa[cur][1]), acc[i][j], 0, 0, 0);
            if constexpr (WIDE) {
              if (i == RT - 1) rdw(w[0], nw, j);               // (its last product of this k-step is on its way)
            }
            __builtin_amdgcn_sched_barrier(0);                 // (hi and lo of an accumulator back to back: 2-4 % less at 323 and 1024 rows)
          }
        }
      }
      sum_left -= KC == 1 ? 2 : 1;
      if (sum_left == 0) {
        sum_left = SUM;
#pragma unroll
        for (int i = 0; i < RT; ++i)
#pragma unroll
          for (int j = 0; j < NW; ++j) {
            tot[i][j] += acc[i][j];
            acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
          }
      }
    }
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
      for (int j = 0; j < NW; ++j) tot[i][j] += acc[i][j];
    // a lane holds row t * 16 + (lane & 15), columns (lane >> 4) * 4 .. + 3 of a slab
    int ln = lane;
    asm volatile("" : "+v"(ln));                               // (keeps the address arithmetic out of the loop)
    typename Epi::template Row<RT> row;
    row.load(epi, J.m0 + t0 * 16 + (ln & 15), J.m1);
#pragma unroll
    for (int i = 0; i < RT; ++i) {
      const int r = J.m0 + (t0 + i) * 16 + (ln & 15);
      if (r < J.m1) {
#pragma unroll
        for (int q = 0; q < NQ; ++q) row.store(epi, i, r, J.split, J.p0 + rd * J.perr + cg + WC * q, (ln >> 4) * 4, tot[i][2 * q], tot[i][2 * q + 1]);
      }
    }
    __builtin_amdgcn_wave_barrier();                           // (lanes meet here, not where the cases below do: what they share stays in scalar registers)
  };
  for (int rd = 0; rd < J.rounds; ++rd) {
    const int nq = (min(J.np - rd * J.perr, J.perr) - cg + WC - 1) / WC;   // pairs cg, cg + WC, ... of the round (at most 0: none)
    // (the fewest row tiles and pairs of a workgroup with such a wave, and the case is compiled only where they can occur)
#define TILE_CASE(R, Q)                                                                                                      \
  case R * 4 + Q:                                                                                                            \
    if constexpr (R <= 8 / WR && (Epi::kWide || R * Q <= kMaxTwo) && KC * 2 * (WR * (R - 1) + 1 + WC * (Q - 1) + 1) <= 8 * CW) {                                 \
      multiply(std::integral_constant<int, R>{}, std::integral_constant<int, Q>{}, rd);                                      \
      break;                                                                                                                 \
    }                                                                                                                        \
    [[fallthrough]];
    switch (rt > 0 && nq > 0 ? rt * 4 + nq : 0) {
      TILE_CASE(1, 1) TILE_CASE(1, 2) TILE_CASE(1, 3)
      TILE_CASE(2, 1) TILE_CASE(2, 2) TILE_CASE(2, 3)
      TILE_CASE(3, 1) TILE_CASE(3, 2) TILE_CASE(3, 3)
      TILE_CASE(4, 1) TILE_CASE(4, 2) TILE_CASE(4, 3)
      default:                                                 // a wave without rows or pairs loads and waits with the others
        for (int st = 0; st < nst; ++st) { top(std::true_type{}); buf = buf + 1 == D ? 0 : buf + 1; }
    }
#undef TILE_CASE
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");            // nothing of this wave is in flight when it ends
}

// k ranges of a launch with `slots` workgroups per row block: as many as leave a workgroup about eight pairs, and no more than
// that where its waves have no room for wide tiles
__host__ __device__ __forceinline__ int tile_splits(int pairs, int ksteps, int slots, int most, bool wide) {
  const int groups = (pairs + 7) / 8, S = wide ? (2 * slots + groups) / (2 * groups) : slots / groups;
  return max(1, min(min(S, most), min(slots, ksteps / 8)));
}

template <typename Epi>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_gemm_tile(const TileGemmArgs a, const Epi epi) {
  extern __shared__ __attribute__((aligned(16))) u32x4_t tile_lds[];
  const int rows = a.n_rows ? min(*a.n_rows, a.rows_cap) : a.rows_cap;
  if (rows <= 0) return;
  // Row blocks: one up to 64 rows, else two or as many as 128 rows each take.  gate/up of the 7B shape, one and two blocks: 64
  // rows 45.6 / 48.9 us, 121 rows 72.6 / 57.4 (the slabs of two workgroups share a fetch from HBM, and 64 rows make stages of
  // two k-steps); 192 rows in two and three blocks 75 / 84, 323 rows in three and four 116 / 120.
  const int RB = rows <= 64 ? 1 : max(2, (rows + 127) / 128);
  const int rows_per = ((rows + RB - 1) / RB + 15) / 16 * 16;
  // consecutive workgroup ids go to the 8 XCDs in turn: logical ids put the row blocks of a column group on one XCD
  const int G = gridDim.x, L = ((int)blockIdx.x & 7) * (G >> 3) + ((int)blockIdx.x >> 3);
  const int slot = L / RB, rb = L - slot * RB;
  const int S = Epi::kSplit ? tile_splits(a.pairs, a.ksteps, G / RB, a.max_splits, Epi::kWide) : 1;
  if (Epi::kSplit && blockIdx.x == 0 && threadIdx.x == 0) *a.splits_out = S;
  const int groups = G / RB / S, split = slot / groups, grp = slot - split * groups;   // (the groups of a k range share A)
  TileJob J;
  J.m0 = rb * rows_per;
  J.m1 = min(rows, J.m0 + rows_per);
  if (split >= S || J.m0 >= J.m1) return;                     // (uniform over the workgroup: nobody is left at a barrier)
  J.nmt = (J.m1 - J.m0 + 15) / 16;
  J.p0 = (int)((long long)a.pairs * grp / groups);
  J.np = (int)((long long)a.pairs * (grp + 1) / groups) - J.p0;
  if (J.np <= 0) return;
  J.split = split;
  J.ks0 = a.ksteps / 8 * split / S * 8;
  J.nks = a.ksteps / 8 * (split + 1) / S * 8 - J.ks0;
  const int most = !Epi::kWide && J.nmt > 4 ? 8 : kMaxPairs;
  J.rounds = (J.np + most - 1) / most;
  J.perr = (J.np + J.rounds - 1) / J.rounds;
  // (the quotients above come out of vector registers)
  for (int* v : {&J.m0, &J.m1, &J.nmt, &J.p0, &J.np, &J.rounds, &J.perr, &J.ks0, &J.nks, &J.split}) *v = __builtin_amdgcn_readfirstlane(*v);
  // a k-step's reads from LDS: 2 x 4 waves read the row tiles four times and the slabs twice, 4 x 2 the other way round
  const bool tall = J.perr <= 6 && J.nmt >= J.perr;
  const int P1 = 2 * (J.nmt + J.perr);                        // pieces per k-step, at most 40
#define TILE_RUN(KC, CW) { if (tall) tile_run<KC, CW, 4>(a, J, epi, tile_lds); else tile_run<KC, CW, 2>(a, J, epi, tile_lds); }
  if (2 * P1 <= 16) TILE_RUN(2, 2)
  else if (2 * P1 <= 24) TILE_RUN(2, 3)
  else if (2 * P1 <= 32) TILE_RUN(2, 4)
  else if (2 * P1 <= 40) TILE_RUN(2, 5)
  else if (P1 <= 24) TILE_RUN(1, 3)
  else if (P1 <= 32) TILE_RUN(1, 4)
  else tile_run<1, 5, 2>(a, J, epi, tile_lds);                // (33 pieces and more: seven pairs at least)
#undef TILE_RUN
}

// 1 / sqrt(mean x^2 + eps) of row r: the pending norm's scalar, applied to the finished sums
__device__ __forceinline__ float tile_row_scale(const float* __restrict__ ssq, int r, int nb, int d, float eps) {
  float ss = 0.f;
  const float* p = ssq + (size_t)r * nb;
  if (nb % 4 == 0) {
    for (int b = 0; b < nb; b += 4) {
      const float4 v = *reinterpret_cast<const float4*>(p + b);
      ss += v.x + v.y + v.z + v.w;
    }
  } else {
    for (int b = 0; b < nb; ++b) ss += p[b];
  }
  return 1.0f / sqrtf(ss / (float)d + eps);
}

// What a launch must hold, checked on the host
inline bool tile_fits(const TileGemmArgs& a, int grid) {
  return grid % 8 == 0 && grid >= a.rows_cap / 128 + 2 && a.ksteps % 8 == 0 && a.ksteps > 0 && a.rows_cap > 0 && a.pairs > 0;
}
template <typename Epi>
hipError_t tile_init() {   // the kernels take more than the default 64 KB of LDS
  return hipFuncSetAttribute((const void*)k_gemm_tile<Epi>, hipFuncAttributeMaxDynamicSharedMemorySize, kTileLds);
}
template <typename Epi>
hipError_t tile_launch(const TileGemmArgs& a, const Epi& e, int grid, hipStream_t s) {
  if (!tile_fits(a, grid)) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_gemm_tile<Epi>, dim3(grid), dim3(512), kTileLds, s, a, e);
  return hipGetLastError();
}

}  // namespace

}  // namespace cerb
