// Geometry shared by the tile GEMM kernels: the 256 x 256 x 64 workgroup tile, its LDS layout and the
// XCD-aware walk of persistent workgroups over the output tiles.
#pragma once
#include "qzo_device.hpp"
#include "qzo_kernels.hpp"

namespace qzo {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));        // as in qzo_nibble.hpp
typedef float floatx16 __attribute__((ext_vector_type(16)));

constexpr int BM = 256, BN = 256, BK = 64;
constexpr int TILE_BYTES = BM * BK * 2;            // 32 KB per operand per stage
constexpr int LDS_BYTES = 4 * TILE_BYTES;          // A0 A1 B0 B1

// Persistent workgroups: the grid is one workgroup per compute unit (or fewer when
// there are fewer tiles) and every workgroup walks a list of output tiles.
// Hardware deals consecutive workgroup ids to the eight XCDs in turn; each XCD
// gets one contiguous eighth of a tile order in which groups of WALK_M M-tiles sweep
// the N-tiles, and its workgroups take consecutive entries of that eighth, so the
// tiles in flight on one XCD share a few A and B row-panels in that XCD's L2.
// M-tiles per group of the walk.  With 32 tiles resident per XCD, groups of 4 (or 2) minimise
// the bytes streamed from HBM (activation panel re-read 6 times, int4 panel 8 times).
constexpr uint32_t WALK_M = 4;
// The walk goes on by additions: a division per tile costs a lone wavefront of a SIMD more than the tile's loads.
struct TileWalk {
  uint32_t tiles_m, tiles_n, id, end, stride;      // entries of the order; this workgroup's next one
  uint32_t first, in;                              // first M-tile of its group, entry within the group
};
__device__ __forceinline__ TileWalk tile_walk_of(uint32_t tiles_m, uint32_t tiles_n, uint32_t wgs) {
  const uint32_t total = tiles_m * tiles_n, per = (total + 7) >> 3, xcd = blockIdx.x & 7u;
  TileWalk w;
  w.tiles_m = tiles_m;
  w.tiles_n = tiles_n;
  w.id = xcd * per + (blockIdx.x >> 3);
  w.end = min((xcd + 1) * per, total);
  w.stride = wgs >> 3;
  const uint32_t width = WALK_M * tiles_n, group = w.id / width;
  w.first = group * WALK_M;
  w.in = w.id - group * width;
  return w;
}
// With K slices (split-K) the walk runs over feature-tiles x slices: entry tn of the walk is feature
// tile tn % real_tiles_n, slice tn / real_tiles_n.
__device__ __forceinline__ TileWalk tile_walk_init(uint32_t M, uint32_t N, uint32_t ksplit = 1) {
  return tile_walk_of((M + BM - 1) / BM, ((N + BN - 1) / BN) * ksplit, gridDim.x);
}
// Tile of the walk's current entry; false when the walk is over.
__device__ __forceinline__ bool tile_walk_get(const TileWalk& w, uint32_t& tm, uint32_t& tn) {
  if (w.id >= w.end) return false;
  static_assert(WALK_M == 4, "group sizes 1 to 4 below");
  const uint32_t gsz = min(w.tiles_m - w.first, WALK_M);
  tn = gsz == 4 ? w.in >> 2 : (gsz == 2 ? w.in >> 1 : (gsz == 1 ? w.in : w.in / 3u));
  tm = w.first + w.in - tn * gsz;
  return true;
}
__device__ __forceinline__ void tile_walk_next(TileWalk& w) {
  w.id += w.stride;
  w.in += w.stride;
  while (w.id < w.end) {
    const uint32_t entries = min(w.tiles_m - w.first, WALK_M) * w.tiles_n;
    if (w.in < entries) break;
    w.in -= entries;
    w.first += WALK_M;
  }
}

__device__ __forceinline__ uint32_t lds_off(uint32_t row, uint32_t chunk) {
  return row * 128u + ((chunk ^ ((row >> 1) & 7u)) << 4);
}

}  // namespace qzo
