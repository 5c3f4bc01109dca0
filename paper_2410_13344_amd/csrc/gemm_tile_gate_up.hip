// The gate/up projection of launches of more than 64 rows on the tile kernel, SwiGLU in its epilogue.
#include "gemm_tile.h"

namespace cerb {

namespace {

// gate and up of the same columns: act = silu(g) * u
struct SwigluEpi {
  static constexpr bool kSplit = false;
  static constexpr bool kRows = false;
  static constexpr bool kWide = true;
  const float* ssq;
  int nb, d, fslabs, Fpad;
  float eps;
  bf16_t* act;
  size_t lo_off;        // row-major planes; 0: fragment order
  __device__ __forceinline__ int slab(int pair, int which) const { return which * fslabs + pair; }
  template <int RT>
  struct Row {
    float rs[RT];
    __device__ __forceinline__ void load(const SwigluEpi& e, int r0, int m1) {
#pragma unroll
      for (int i = 0; i < RT; ++i) rs[i] = tile_row_scale(e.ssq, min(r0 + i * 16, m1 - 1), e.nb, e.d, e.eps);
    }
    __device__ __forceinline__ void store(const SwigluEpi& e, int i, int r, int split, int pair, int c, const f32x4_t& g4, const f32x4_t& u4) const {
      float o[4];
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const float g = g4[v] * rs[i], u = u4[v] * rs[i];
        o[v] = g / (1.0f + expf(-g)) * u;
      }
      const int col = pair * 16 + c;
      if (e.lo_off) {
        st_a4(e.act + (size_t)r * e.Fpad + col, e.lo_off, o);
        return;
      }
      // in fragment order columns col .. col + 3 are half of a 16-byte piece
      union { bf16_t h[4]; uint2 u; } hi, lo;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        hi.h[v] = f32_to_bf16(o[v]);
        lo.h[v] = f32_to_bf16(o[v] - bf16_to_f32(hi.h[v]));
      }
      unsigned char* f = reinterpret_cast<unsigned char*>(e.act) + ((size_t)(r >> 4) * (e.Fpad >> 5) + (col >> 5)) * 2048 + ((r & 15) + 16 * ((col & 31) >> 3)) * 16 + (col & 7) * 2;
      *reinterpret_cast<uint2*>(f) = hi.u;
      *reinterpret_cast<uint2*>(f + 1024) = lo.u;
    }
  };
};

}  // namespace

hipError_t init_tile_gate_up() { return tile_init<SwigluEpi>(); }

hipError_t launch_tile_gate_up(const TileGemmArgs& a, const FusedGateUpArgs& g, int grid, hipStream_t s) {
  return tile_launch(a, SwigluEpi{g.ssq, g.nb, g.d, a.pairs, g.Fpad, g.eps, g.act, g.lo_off}, grid, s);
}

}  // namespace cerb
