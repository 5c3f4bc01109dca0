// Whole-K GEMMs with fused epilogues for launches of more than 64 rows (bf16 mode): the gate/up projection with SwiGLU.
//
// A workgroup of 8 waves per compute unit owns a row block (at most 128 rows) and a few 16-column slabs over the full K, so
// there are no partial planes: the epilogue works on finished sums and no consumer kernel follows.  Row blocks and column
// groups are formed on the device from the step's row count (the host knows a bound only): the fewest row blocks of at most
// 128 rows, two above 64 rows; the slabs, in pairs whose columns an epilogue needs together, are dealt evenly to the
// workgroups of a row block; what does not fit the accumulators (12 pairs) goes in rounds.
//
// Both operands go global -> LDS by direct loads in MFMA fragment order, several stages deep, and are shared: the waves
// stand 2 x 4, half of the row tiles by every fourth pair, so a fragment of A is read by four waves and one of W by two.  The
// fragments of the next k-step are read from LDS while this one is multiplied, across the barrier between stages too (a
// stage has landed for everyone one barrier before its turn).  What that is worth, gate/up of the 7B shape (K = 4096,
// N = 22016), bare kernel: 323 rows 149 us with the reads in front of the products, 116 with them a k-step ahead; 121 rows
// 71 and 57; 1024 rows 330 and 306.  A stage is 40 pieces of 1 KB at most; small tiles take two k-steps per stage (121 rows
// 57 us, with one 71).  Bounds: up to about 256 rows what the L2s and HBM deliver into a compute unit (128 rows x 4096 x
// 4 bytes of A and the slabs come in at 13-15 TB/s over the chip, 53 us of the 57 at 121 rows); above that the matrix cores
// at the clock the load leaves them (1024 rows without any loads: 250-265 us).
//
// The products are W A^T: a lane then holds four consecutive columns of one row, which go out as one store per plane.
#include <type_traits>

#include "step_kernels.h"

namespace cerb {

namespace {

constexpr int kTileLds = 160 * 1024;
constexpr int kMaxPairs = 12;   // slab pairs of a round: 3 per wave

__device__ __forceinline__ void tile_dma16(const char* p, unsigned lds_addr) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds_addr), "v"(p) : "memory", "m0");
}

// Row tiles [m0/16, m0/16 + nmt) by pairs [p0, p0 + np) of the launch
struct TileJob { int m0, m1, nmt, p0, np, rounds, perr; };

// KC k-steps per stage, CW pieces of 1 KB per wave and stage
template <int KC, int CW, typename Epi>
__device__ __forceinline__ void tile_run(const TileGemmArgs& a, const TileJob& J, const Epi& epi, u32x4_t* lds) {
  constexpr unsigned SB = CW * 8 * 1024;
  constexpr int D = kTileLds / (int)SB;                        // stages in LDS
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int nst = a.ksteps / KC;
  const int rg = wave >> 2, cg = rg ? 7 - wave : wave;         // (the two waves of a SIMD: the pairs of cg and of 3 - cg)
  const int rt = rg ? J.nmt / 2 : (J.nmt + 1) / 2, t0 = rg ? (J.nmt + 1) / 2 : 0;
  const int P1 = 2 * J.nmt + 2 * J.perr;                       // pieces per k-step: A (row tile, plane), then W (pair, slab)
  const unsigned ldsb = (unsigned)(unsigned long)((__attribute__((address_space(3))) const unsigned char*)lds);

  // ---- pieces q * 8 + wave of a stage (past the last one: that one once more, into a slot nobody reads)
  const char* src[CW];
  unsigned step[CW];
  auto bases = [&](int rd) {
#pragma unroll
    for (int q = 0; q < CW; ++q) {
      const int p = min(q * 8 + wave, KC * P1 - 1), kc = p / P1, r = p - kc * P1;
      if (r < 2 * J.nmt) {
        src[q] = reinterpret_cast<const char*>(a.A) + lane * 16 + ((size_t)((size_t)(J.m0 / 16 + (r >> 1)) * a.ksteps + kc) * 2 + (r & 1)) * 1024;
        step[q] = KC * 2048;
      } else {
        const int pos = r - 2 * J.nmt, pair = min(J.p0 + rd * J.perr + (pos >> 1), J.p0 + J.np - 1);
        src[q] = reinterpret_cast<const char*>(a.W) + lane * 16 + ((size_t)epi.slab(pair, pos & 1) * a.ksteps + kc) * 1024;
        step[q] = KC * 1024;
      }
    }
  };
  bases(0);
  int ist = 0, ird = 0, ibuf = 0, left = nst * J.rounds;       // the stage to be issued; issues past the last repeat it
  auto issue = [&]() {
    const unsigned l0 = __builtin_amdgcn_readfirstlane(ldsb + ibuf * SB + wave * 1024);
#pragma unroll
    for (int q = 0; q < CW; ++q) tile_dma16(src[q], l0 + q * 8192);
    ibuf = ibuf + 1 == D ? 0 : ibuf + 1;
    if (left > 1) {
      --left;
      if (++ist == nst) {
        ist = 0;
        bases(++ird);
      } else {
#pragma unroll
        for (int q = 0; q < CW; ++q) src[q] += step[q];
      }
    }
  };
#pragma unroll
  for (int i = 0; i < D - 1; ++i) issue();

  int buf = 0;
  // Top of stage n: this wave's pieces of stage n + 1 have landed, then everyone's; and everyone has multiplied stage n - 1,
  // whose buffer takes stage n + D - 1 (no lgkmcnt: a read that still runs here is one of stage n's first fragments).
  auto top = [&]() {
    asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"((D - 3) * CW) : "memory");
    issue();
  };
  auto multiply = [&](auto rtc, auto nqc, int rd) {
    constexpr int RT = decltype(rtc)::value, NQ = decltype(nqc)::value, NW = 2 * NQ;
    const u32x4_t* la = lds + lane + t0 * 128;
    const u32x4_t* lw = lds + lane + (2 * J.nmt + cg * 2) * 64;
    typename Epi::template Row<RT> row;
    row.load(epi, J.m0 + t0 * 16 + (lane & 15), J.m1);
    f32x4_t acc[RT][NW];
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
      for (int j = 0; j < NW; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    u32x4_t w[2][NW], fa[2][2];                                // this k-step's slabs and the next one's; a row tile and the next
    auto rdw = [&](u32x4_t (&d)[NW], const u32x4_t* s, int j) { d[j] = s[(j >> 1) * 512 + (j & 1) * 64]; };
    const unsigned p1 = P1 * 64;
    for (int st = 0; st < nst; st += (KC == 1 ? 2 : 1)) {      // two k-steps per trip
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        if (KC == 1 || h == 0) top();
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
#pragma unroll
          for (int j = i * NW / RT; j < (i + 1) * NW / RT; ++j) rdw(w[h ^ 1], nw, j);
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int j = 0; j < NW; ++j) {
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, w[h][j]), __builtin_bit_cast(bf16x8_t, fa[cur][0]), acc[i][j], 0, 0, 0);
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, w[h][j]), __builtin_bit_cast(bf16x8_t, fa[cur][1]), acc[i][j], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);                 // (hi and lo of an accumulator back to back: 2-4 % less at 323 and 1024 rows)
          }
        }
      }
    }
    // a lane holds row t * 16 + (lane & 15), columns (lane >> 4) * 4 .. + 3 of a slab
    int ln = lane;
    asm volatile("" : "+v"(ln));                               // (keeps the address arithmetic out of the loop)
#pragma unroll
    for (int i = 0; i < RT; ++i) {
      const int r = J.m0 + (t0 + i) * 16 + (ln & 15);
      if (r < J.m1) {
#pragma unroll
        for (int q = 0; q < NQ; ++q) row.store(epi, i, r, J.p0 + rd * J.perr + cg + 4 * q, (ln >> 4) * 4, acc[i][2 * q], acc[i][2 * q + 1]);
      }
    }
  };
  for (int rd = 0; rd < J.rounds; ++rd) {
    const int nq = (min(J.np - rd * J.perr, J.perr) - cg + 3) >> 2;   // pairs cg, cg + 4, cg + 8 of the round (at most 0: none)
#define TILE_CASE(R, Q)                                                                                                      \
  case R * 4 + Q:                                                                                                            \
    if constexpr (KC * (2 * (2 * R - 1) + 2 * (4 * Q - 3)) <= 8 * CW) {                                                      \
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
        for (int st = 0; st < nst; ++st) { top(); buf = buf + 1 == D ? 0 : buf + 1; }
    }
#undef TILE_CASE
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");            // nothing of this wave is in flight when it ends
}

template <typename Epi>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_gemm_tile(const TileGemmArgs a, const Epi epi) {
  extern __shared__ __attribute__((aligned(16))) u32x4_t tile_lds[];
  const int rows = min(*a.n_rows, a.rows_cap);
  if (rows <= 0) return;
  // Row blocks: one up to 64 rows, else two or as many as 128 rows each take.  gate/up of the 7B shape, one and two blocks: 64
  // rows 45.6 / 48.9 us, 121 rows 72.6 / 57.4 (the slabs of two workgroups share a fetch from HBM, and 64 rows make stages of
  // two k-steps); 192 rows in two and three blocks 75 / 84, 323 rows in three and four 116 / 120.
  const int RB = rows <= 64 ? 1 : max(2, (rows + 127) / 128);
  const int rows_per = ((rows + RB - 1) / RB + 15) / 16 * 16;
  // consecutive workgroup ids go to the 8 XCDs in turn: logical ids put the row blocks of a column group on one XCD
  const int G = gridDim.x, L = ((int)blockIdx.x & 7) * (G >> 3) + ((int)blockIdx.x >> 3);
  const int groups = G / RB, grp = L / RB, rb = L - grp * RB;
  TileJob J;
  J.m0 = rb * rows_per;
  J.m1 = min(rows, J.m0 + rows_per);
  if (grp >= groups || J.m0 >= J.m1) return;                  // (uniform over the workgroup: nobody is left at a barrier)
  J.nmt = (J.m1 - J.m0 + 15) / 16;
  J.p0 = (int)((long long)a.pairs * grp / groups);
  J.np = (int)((long long)a.pairs * (grp + 1) / groups) - J.p0;
  if (J.np <= 0) return;
  J.rounds = (J.np + kMaxPairs - 1) / kMaxPairs;
  J.perr = (J.np + J.rounds - 1) / J.rounds;
  const int P1 = 2 * (J.nmt + J.perr);                        // at most 40
  if (2 * P1 <= 32) tile_run<2, 4>(a, J, epi, tile_lds);
  else if (2 * P1 <= 40) tile_run<2, 5>(a, J, epi, tile_lds);
  else if (P1 <= 24) tile_run<1, 3>(a, J, epi, tile_lds);
  else if (P1 <= 32) tile_run<1, 4>(a, J, epi, tile_lds);
  else tile_run<1, 5>(a, J, epi, tile_lds);
}

// gate and up of the same columns: act = silu(g) * u, the pending norm's scalar applied to both
struct SwigluEpi {
  const float* ssq;
  int nb, d, fslabs, Fpad;
  float eps;
  bf16_t* act;
  size_t lo_off;
  __device__ __forceinline__ int slab(int pair, int which) const { return which * fslabs + pair; }
  template <int RT>
  struct Row {
    float rs[RT];
    __device__ __forceinline__ void load(const SwigluEpi& e, int r0, int m1) {
#pragma unroll
      for (int i = 0; i < RT; ++i) {
        const int r = min(r0 + i * 16, m1 - 1);
        float ss = 0.f;
        for (int b = 0; b < e.nb; ++b) ss += e.ssq[(size_t)r * e.nb + b];
        rs[i] = 1.0f / sqrtf(ss / (float)e.d + e.eps);
      }
    }
    __device__ __forceinline__ void store(const SwigluEpi& e, int i, int r, int pair, int c, const f32x4_t& g4, const f32x4_t& u4) const {
      float o[4];
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const float g = g4[v] * rs[i], u = u4[v] * rs[i];
        o[v] = g / (1.0f + expf(-g)) * u;
      }
      st_a4(e.act + (size_t)r * e.Fpad + pair * 16 + c, e.lo_off, o);
    }
  };
};

}  // namespace

hipError_t init_tile_gemm() {   // the kernels take more than the default 64 KB of LDS
  return hipFuncSetAttribute((const void*)k_gemm_tile<SwigluEpi>, hipFuncAttributeMaxDynamicSharedMemorySize, kTileLds);
}

hipError_t launch_tile_gate_up(const TileGemmArgs& a, const FusedGateUpArgs& g, int grid, hipStream_t s) {
  if (grid % 8 || grid < a.rows_cap / 128 + 2 || a.ksteps % 8) return hipErrorInvalidValue;
  const SwigluEpi e{g.ssq, g.nb, g.d, a.pairs, g.Fpad, g.eps, g.act, g.lo_off};
  hipLaunchKernelGGL(k_gemm_tile<SwigluEpi>, dim3(grid), dim3(512), kTileLds, s, a, e);
  return hipGetLastError();
}

}  // namespace cerb
