// The QKV projection of launches of more than 128 rows on the tile kernel, RoPE and the KV write in its epilogue.
#include "gemm_tile.h"

namespace cerb {

namespace {

// Pairs, in this order: columns j .. j + 15 and j + dh/2 .. of a q head (RoPE rotates one with the other), the same of the k
// heads, two neighbouring v slabs
struct RopeEpi {
  static constexpr bool kSplit = false;
  static constexpr bool kRows = false;
  static constexpr bool kWide = false;
  FusedQkvArgs f;
  __device__ __forceinline__ int slab(int pair, int which) const {
    const int spd = f.D.d / 16, sph = f.D.dh / 16, sec = pair / (spd / 2), t = pair - sec * (spd / 2);
    return sec * spd + (sec == 2 ? 2 * t + which : t / (sph / 2) * sph + t % (sph / 2) + which * (sph / 2));
  }
  template <int RT>
  struct Row {
    float rs[RT];
    int seq[RT], crow[RT];     // sequence and cache row
    __device__ __forceinline__ void load(const RopeEpi& e, int r0, int m1) {
#pragma unroll
      for (int i = 0; i < RT; ++i) {
        const int r = min(r0 + i * 16, m1 - 1);
        rs[i] = tile_row_scale(e.f.ssq, r, e.f.nb, e.f.D.d, e.f.D.eps);
        seq[i] = e.f.rm.row_seq[r];
        crow[i] = e.f.rm.seq_L[seq[i]] + e.f.rm.row_node[r];
      }
    }
    __device__ __forceinline__ void store(const RopeEpi& e, int i, int r, int split, int pair, int c, const f32x4_t& a4, const f32x4_t& b4) const {
      const Dims& D = e.f.D;
      const int s0 = e.slab(pair, 0), d = D.d, dh = D.dh, sec = s0 / (d / 16);
      const int col = s0 * 16 - sec * d + c, h = col / dh, j = col - h * dh, gap = sec == 2 ? 16 : dh / 2;   // first column of a4; b4: gap later
      float y0[4], y1[4];
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const float x0 = a4[v] * rs[i], x1 = b4[v] * rs[i];
        y0[v] = x0;
        y1[v] = x1;
        if (sec < 2) {
          const float2 rot = e.f.rope_cs[(size_t)r * (dh / 2) + j + v];
          y0[v] = x0 * rot.x - x1 * rot.y;
          y1[v] = x0 * rot.y + x1 * rot.x;
        }
      }
      bf16_t *const planes_q = e.f.q, *const planes_k = e.f.ktree, *const planes_v = e.f.vtree;   // (selected by value: by address the arguments would go through scratch)
      bf16_t* plane = (sec == 0 ? planes_q : sec == 1 ? planes_k : planes_v) + (size_t)r * d + col;
      st_a4(plane, e.f.lo_off, y0);
      st_a4(plane + gap, e.f.lo_off, y1);
      if (sec > 0 && e.f.kv_layer) {   // (the benchmark hook has no cache to write to)
        bf16_t* cr = e.f.kv_layer + (((size_t)((sec - 1) * D.Bmax + seq[i]) * D.nH + h) * D.cap + crow[i]) * dh + j;
        union { bf16_t h[4]; uint2 u; } k0, k1;
#pragma unroll
        for (int v = 0; v < 4; ++v) { k0.h[v] = f32_to_bf16(y0[v]); k1.h[v] = f32_to_bf16(y1[v]); }
        *reinterpret_cast<uint2*>(cr) = k0.u;
        *reinterpret_cast<uint2*>(cr + gap) = k1.u;
      }
    }
  };
};

}  // namespace

hipError_t init_tile_qkv() { return tile_init<RopeEpi>(); }

hipError_t launch_tile_qkv(const TileGemmArgs& a, const FusedQkvArgs& f, int grid, hipStream_t s) {
  return f.D.d % 32 ? hipErrorInvalidValue : tile_launch(a, RopeEpi{f}, grid, s);
}

}  // namespace cerb
