// Binning by tile (tiles.hip): what the binning entry points use of it.
#pragma once

#include "common.hpp"

namespace msplat {

constexpr int32_t kTableTiles = 2048;      // tiles of a count / place workgroup's LDS table (8 KB)
constexpr int32_t kTileRecords = 256;      // records of such a workgroup
constexpr int32_t kSampleGroups = 64;      // groups of that many records that the choice of path looks at
constexpr int32_t kOrderTiles = 1024;      // tiles per group of the processing order
constexpr int32_t kMaxOrderGroups = 512;   // at most 524,288 tiles
constexpr int32_t kLengthBuckets = 33;     // bit lengths of a list length
constexpr int32_t kShortCap = 512;         // list lengths of the sort kernels (tiles.hip)
constexpr int32_t kMidCap = 2048;
constexpr int32_t kLongCap = 8192;         // entries a workgroup sorts at once, at most
constexpr int32_t kSliceKeys = 4096;       // aimed entries of a longer list's slice
constexpr int32_t kSample = 1024;          // entries that bound the slices
constexpr int32_t kMaxSlices = 1 << 16;    // slices over all lists
constexpr int32_t kTileMaxList = 65536;    // longer lists: the radix sort
constexpr int kTileStats = 7;              // n_isect, n_visible, zmin, zmax, longest list, slices, pairs by tile

// Workgroups that sort a list of more than kMidCap entries (0: a shorter one).
__host__ __device__ inline uint32_t slices_of(uint32_t len) {
  if (len <= (uint32_t)kMidCap) return 0u;
  return len <= (uint32_t)kLongCap ? 1u : (len + (uint32_t)kSliceKeys - 1u) / (uint32_t)kSliceKeys;
}

struct TileWs {
  uint32_t* sum;     // [workgroups] pairs, then their exclusive scan
  uint32_t* zmin;    // [workgroups]
  uint32_t* zmax;    // [workgroups]
  uint32_t* vis;     // [workgroups]
  uint64_t* stats;   // [kTileStats]
  uint32_t* hist;    // [groups][kLengthBuckets]
  uint8_t* bucket;   // [tiles] length bucket
  uint4* sample;     // [kSampleGroups] (tiles of the rectangle, pairs, tiles of the largest box, -)
  uint2* slices;     // [kMaxSlices] (tile, slice) of the lists of more than kMidCap entries
};

size_t tile_ws_bytes(int64_t nrec);
TileWs carve_tiles(void* ws, int64_t nrec);
bool tiles_eligible(const ViewSet& vs);
int32_t count_by_tile(const gs_projected_t* proj, const ViewSet& vs, int32_t V, int64_t n, uint32_t* ranges,
                      const TileWs& ws, uint64_t* host, hipStream_t s);
int32_t offsets_by_tile(const gs_projected_t* proj, const ViewSet& vs, int32_t V, int64_t n, const TileWs& ws,
                        uint32_t* offsets, uint32_t* tile_order, hipStream_t s);
bool lists_by_tile_pay(const gs_bin_stats_t* stats);
int32_t lists_by_tile(const gs_projected_t* proj, const ViewSet& vs, int32_t V, int64_t n,
                      const gs_bin_stats_t* stats, const TileWs& ws, uint32_t* ranges, uint64_t* keys, uint32_t* vals,
                      void* sort_ws, hipStream_t s);

}  // namespace msplat
