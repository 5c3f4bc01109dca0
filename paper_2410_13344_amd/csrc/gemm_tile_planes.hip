// The O and down projections of launches of more than 128 rows on the tile kernel: fp32 planes over ranges of K.
#include "gemm_tile.h"

namespace cerb {

namespace {

// fp32 planes, one per k range, for the consumer to sum.  ROWS: A is row-major, with the addresses of its lanes in vector registers
template <bool ROWS>
struct PlaneEpi {
  static constexpr bool kSplit = true, kRows = ROWS, kWide = !ROWS;
  float* out;
  size_t pstride;
  int N;
  __device__ __forceinline__ int slab(int pair, int which) const { return pair * 2 + which; }
  template <int RT>
  struct Row {
    __device__ __forceinline__ void load(const PlaneEpi&, int, int) {}
    __device__ __forceinline__ void store(const PlaneEpi& e, int, int r, int split, int pair, int c, const f32x4_t& a4, const f32x4_t& b4) const {
      float* o = e.out + split * e.pstride + (size_t)r * e.N + pair * 32 + c;
      *reinterpret_cast<f32x4_t*>(o) = a4;
      *reinterpret_cast<f32x4_t*>(o + 16) = b4;
    }
  };
};

}  // namespace

hipError_t init_tile_planes() {
  const hipError_t e = tile_init<PlaneEpi<false>>();
  return e == hipSuccess ? tile_init<PlaneEpi<true>>() : e;
}

int tile_plane_splits(int pairs, int ksteps, int grid, int most, bool rows) { return tile_splits(pairs, ksteps, grid, most, !rows); }

hipError_t launch_tile_planes(const TileGemmArgs& a, float* out, size_t pstride, int grid, hipStream_t s) {
  if (a.max_splits < 1 || !a.splits_out || pstride % 4) return hipErrorInvalidValue;
  if (a.lda) return tile_launch(a, PlaneEpi<true>{out, pstride, a.pairs * 32}, grid, s);
  return tile_launch(a, PlaneEpi<false>{out, pstride, a.pairs * 32}, grid, s);
}

}  // namespace cerb
