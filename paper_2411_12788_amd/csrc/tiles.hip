// a2-a4 by tile: the sorted lists without sorting pairs across the image.
//
// A list holds, for one tile, the records whose boxes meet it, by (depth,
// record index).  That order is total, so it does not matter in which order
// the pairs of a tile arrive:
//   1. k_tile_count    pairs per tile (LDS histograms, one global add per tile
//                      and workgroup), statistics and pair totals per workgroup
//   2. k_tile_scan     list starts, longest list, totals
//   3. k_tile_offsets  offsets of the records, and the tile processing order
//                      (while the totals travel to the host)
//   4. k_tile_place    every pair as one 8-byte entry (depth | record) in its
//                      tile's run (room taken per workgroup and tile)
//   5. k_tile_sort     each run sorted in LDS, record indices written
// The radix sort of (tile | depth) keys moves every pair through memory about
// sixteen times (five to six passes of an up-sweep and a scatter) in nineteen
// launches; here a pair is written once and read once (in lists of more than
// kLongCap entries once per slice).  Lists longer than kTileMaxList, scenes that
// are not in spatial order or whose boxes all cover the view (k_tile_start), and
// records whose own counts are not what their boxes give go to the radix sort.
#include "common.hpp"
#include "tiles.hpp"

namespace msplat {

constexpr int kWaves = kBlock / kWave;

// ---------------------------------------------------------------------------
// the tiles of a record
// ---------------------------------------------------------------------------
// Calls f(tile column, tile row, depth bits, record of the view) for every pair
// of the wave's records (one per lane, w > 0 where there is one) in tile rows
// [row0, row0 + rows).  Boxes hold
// from one tile to the whole image, so the lanes do not walk their own: the
// tiles of all boxes of less than kWideTiles form one run that the wave takes
// 64 at a time.  Lane l of a turn takes tile c0 + l; its record is the last one
// that starts at or before it, found from the marks that the records starting
// inside the turn leave.  Larger boxes fill whole turns and are taken one by
// one.  With tile culling a record that lost tiles (w < box) is tested per
// tile, as the projection did when it counted them.  Only a box's part in those
// rows is walked: with all of it walked for each band of rows and the tiles
// outside dropped, 256 Gaussians over all of a 4096x4096 view were binned in
// 396 ms.
constexpr uint32_t kWideTiles = 64;
constexpr uint32_t kTested = 0x80000000u;

template <bool CULL>
struct WalkLds {  // of one wave
  uint32_t start[2 * kWave];  // first tile of each record, then 0xffffffff
  uint4 rec[kWave];           // box x, box y, depth bits, record (| kTested)
  uint32_t mark[kWave];       // 0 between turns
  float4 r0[CULL ? kWave : 1], r1[CULL ? kWave : 1];
};
__device__ __forceinline__ uint32_t lanes_below(uint64_t m) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}
// Inclusive sum over the wave (row shifts, then the row broadcasts).
__device__ __forceinline__ uint32_t wave_scan_u32(uint32_t x) {
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xF, 0xF, false);
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xF, 0xF, false);
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xF, 0xF, false);
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xF, 0xF, false);
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xA, 0xF, false);
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xC, 0xF, false);
  return x;
}
__device__ __forceinline__ uint32_t last_lane(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_readlane((int)x, kWave - 1);
}
// Largest value of the wave.
__device__ __forceinline__ uint32_t wave_top_u32(uint32_t x) {
  auto up = [](uint32_t a, uint32_t b) { return a > b ? a : b; };
  x = up(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xF, 0xF, false));
  x = up(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xF, 0xF, false));
  x = up(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xF, 0xF, false));
  x = up(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xF, 0xF, false));
  x = up(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xA, 0xF, false));
  x = up(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xC, 0xF, false));
  return last_lane(x);
}

template <bool CULL, typename F>
__device__ __forceinline__ void for_each_tile(WalkLds<CULL>& L, int4 b, int64_t r, uint32_t i,
                                              const float* __restrict__ rec, float tile_cull, int32_t row0,
                                              int32_t rows, F&& f) {
  const int lane = (int)lane_id();
  auto first_row = [&](uint32_t by) { return max((int32_t)((by & 0xffffu) >> 4), row0); };
  auto rows_here = [&](uint32_t by) { return max(min((int32_t)(by >> 20), row0 + rows - 1) - first_row(by) + 1, 0); };
  auto columns = [&](uint32_t bx) { return (int32_t)(bx >> 20) - (int32_t)((bx & 0xffffu) >> 4) + 1; };
  uint32_t area = 0, whole = 0;
  if (b.w > 0) {
    const int32_t nx = columns((uint32_t)b.x);
    whole = (uint32_t)(nx * ((int32_t)((uint32_t)b.y >> 20) - (int32_t)(((uint32_t)b.y & 0xffffu) >> 4) + 1));
    area = (uint32_t)(nx * rows_here((uint32_t)b.y));
  }
  const uint64_t some = __builtin_amdgcn_ballot_w64(area > 0);
  if (some == 0ull) return;
  const uint64_t narrow = __builtin_amdgcn_ballot_w64(area > 0 && area < kWideTiles);
  const uint32_t run = area < kWideTiles ? area : 0u;
  const uint32_t incl = wave_scan_u32(run), total = last_lane(incl);
  const uint32_t count = (uint32_t)__popcll(narrow);
  // the run's records first, then the wide ones
  const uint32_t slot = area < kWideTiles ? lanes_below(narrow) : count + lanes_below(some & ~narrow);
  wave_sync();
  L.mark[lane] = 0u;
  L.start[kWave + lane] = 0xffffffffu;
  L.start[lane] = 0xffffffffu;
  wave_sync();
  if (area > 0) {
    const bool test = CULL && (uint32_t)b.w < whole;
    if (area < kWideTiles) L.start[slot] = incl - area;
    L.rec[slot] = make_uint4((uint32_t)b.x, (uint32_t)b.y, (uint32_t)b.z, i | (test ? kTested : 0u));
    if (test) {
      const float4* R4 = reinterpret_cast<const float4*>(rec + r * kRecFloats);
      L.r0[CULL ? slot : 0] = R4[0];
      L.r1[CULL ? slot : 0] = R4[1];
    }
  }
  wave_sync();
  auto visit = [&](uint32_t own, uint32_t local) {
    const uint4 e = L.rec[own];
    const int32_t x0 = (int32_t)(e.x & 0xffffu), x1 = (int32_t)(e.x >> 16);
    const int32_t y0 = (int32_t)(e.y & 0xffffu), y1 = (int32_t)(e.y >> 16);
    const uint32_t nx = (uint32_t)columns(e.x);
    // local / nx: the quotient's distance from a whole number is at least
    // 0.5 / nx, above the reciprocal's error for boxes of up to 2M tiles
    const uint32_t dy = (uint32_t)(((float)local + 0.5f) * __builtin_amdgcn_rcpf((float)nx));
    const int32_t tx = (x0 >> 4) + (int32_t)(local - dy * nx), ty = first_row(e.y) + (int32_t)dy;
    bool keep = true;
    if (CULL && (e.w & kTested))
      keep = tile_kept(L.r0[CULL ? own : 0], L.r1[CULL ? own : 0], tx, ty, x0, x1, y0, y1, tile_cull);
    if (keep) f(tx, ty, e.z, e.w & ~kTested);
  };
  uint32_t own0 = 0;
  for (uint32_t c0 = 0; c0 < total; c0 += kWave) {
    // records after own0 start at c0 or later
    const uint32_t nxt = L.start[own0 + 1 + lane] - c0;
    if (nxt < (uint32_t)kWave) L.mark[nxt] = 1u;
    wave_sync();
    const uint64_t m = __builtin_amdgcn_ballot_w64(L.mark[lane] != 0u);
    wave_sync();
    if (nxt < (uint32_t)kWave) L.mark[nxt] = 0u;
    wave_sync();
    const uint32_t t = c0 + (uint32_t)lane;
    const uint32_t own = own0 + lanes_below(m) + (uint32_t)((m >> lane) & 1ull);
    if (t < total) visit(own, t - L.start[own]);
    own0 += (uint32_t)__popcll(m);
  }
  const uint32_t all = (uint32_t)__popcll(some);
  for (uint32_t q = count; q < all; ++q) {
    const uint4 e = L.rec[q];
    const uint32_t tiles = (uint32_t)(columns(e.x) * rows_here(e.y));
#pragma unroll 2
    for (uint32_t t = lane; t < tiles; t += kWave) visit(q, t);
  }
}

// Workgroup (x, y): records [x kPer, x kPer + kPer) of view y, dealt to its
// waves in turn (records with large boxes sit together).  Its table in LDS
// covers the rectangle of tiles that its records meet, which the spatial order
// keeps small (a table of the whole view, cleared and read by every workgroup,
// took more time than the pairs); a rectangle of more tiles than the table
// holds is taken in bands of rows.  256 records: at 3M records 512 are as fast
// and 1,024 slower, at 200k they take 1.4 and 2.2 times as long (large boxes
// sit together, small workgroups even them out); 2,048 tiles: twice and four
// times that hold fewer workgroups a CU and are up to 10 % slower.
struct TileArgs {
  const int4* bin;
  const float* rec;
  float tile_cull;
  int64_t n;
  int32_t table;  // words of the table
};
constexpr int kPer = kTileRecords;
static_assert(kPer == kBlock, "one record per thread");

struct TileRect {
  int32_t x0, y0, w, h;
};
struct RectLds {
  uint32_t v[4][kWaves];
};
// (Clamped to the view, so that no record can lead outside the table.)
__device__ __forceinline__ TileRect block_rect(RectLds& s, int4 b, int32_t tiles_x, int32_t tiles_y) {
  uint32_t t[4] = {0u, 0u, 0u, 0u};  // ~first and last tile column, then row; 0 without a record
  if (b.w > 0) {
    t[0] = 0xffffu - (((uint32_t)b.x & 0xffffu) >> 4);
    t[1] = (uint32_t)b.x >> 20;
    t[2] = 0xffffu - (((uint32_t)b.y & 0xffffu) >> 4);
    t[3] = (uint32_t)b.y >> 20;
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    t[k] = wave_top_u32(t[k]);
    if (lane_id() == 0) s.v[k][threadIdx.x / kWave] = t[k];
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 4; ++k) {
#pragma unroll
    for (int q = 0; q < kWaves; ++q) t[k] = s.v[k][q] > t[k] ? s.v[k][q] : t[k];
    t[k] = uniform_u32(t[k]);
  }
  TileRect r;
  r.x0 = (int32_t)(0xffffu - t[0]);
  r.y0 = (int32_t)(0xffffu - t[2]);
  const int32_t x1 = (int32_t)t[1] < tiles_x ? (int32_t)t[1] : tiles_x - 1;
  const int32_t y1 = (int32_t)t[3] < tiles_y ? (int32_t)t[3] : tiles_y - 1;
  if (t[0] == 0u || x1 < r.x0 || y1 < r.y0) return TileRect{0, 0, 0, 0};  // no records
  r.w = x1 - r.x0 + 1;
  r.h = y1 - r.y0 + 1;
  return r;
}
__device__ __forceinline__ int64_t record_of(int64_t first) {
  return first + (int64_t)lane_id() * kWaves + threadIdx.x / kWave;
}
__device__ __forceinline__ int4 load_record(const TileArgs& a, int v, int64_t i) {
  return i < a.n ? a.bin[(int64_t)v * a.n + i] : make_int4(0, 0, 0, 0);
}
// Calls f(table index, depth bits, record) for the pairs of rows [y0, y0 + rows)
// of the rectangle.
template <bool CULL, typename F>
__device__ __forceinline__ void walk_rows(WalkLds<CULL>& L, const TileArgs& a, int v, int64_t i, int4 b,
                                          const TileRect& r, int32_t y0, int32_t rows, F&& f) {
  for_each_tile(L, b, (int64_t)v * a.n + i, (uint32_t)i, a.rec, a.tile_cull, y0, rows,
                [&](int32_t tx, int32_t ty, uint32_t z, uint32_t who) {
                  const int32_t row = ty - y0, col = tx - r.x0;
                  if ((uint32_t)row < (uint32_t)rows && (uint32_t)col < (uint32_t)r.w) f(row * r.w + col, z, who);
                });
}

// ---------------------------------------------------------------------------
// 0. start
// ---------------------------------------------------------------------------
// Clears the ranges, and measures on kSampleGroups groups of kPer records how
// many tiles a workgroup's rectangle has per pair.  In a scene that is not in
// spatial order it is the whole view: nearly every pair then needs its own
// global add, and the radix sort is faster.  Project and binning at 1080p, in
// spatial and in random order: 3M records, 4.6M pairs 378 and 897 us by tile,
// 465 and 476 us by radix sort (0.3 and 21 tiles per pair); 8.7M pairs 448 and
// 1,041 against 623 and 678 us (11 per pair); 500k records, 1.2M pairs 99 and
// 223 against 193 and 200 us (6.5); 200k records 87 and 127 against 156 and
// 153 us (5).
// The other end is a group whose boxes are nearly all as large as the largest:
// a group's pairs are one workgroup's work here (1.3 ns a pair for the three
// walks) and a record's boxes one thread's in the radix sort's emission (0.16 us
// a tile of the largest box), so the radix sort is faster above 128 times the
// largest box.  512 records over all of a 1920x1080 view 2.74 ms by tile and
// 1.55 by radix sort, 64 of them 0.77 and 1.45, 256 of them beside 4,096 small
// ones 0.53 and 1.62.  Below kMostGroupPairs both take much the same (256 over
// a 256x256 view: 156 and 157 us).
constexpr uint64_t kTilesPerTwoPairs = 11;
constexpr uint32_t kMostGroupPairs = 1u << 16, kMostBoxes = 128;

__global__ __launch_bounds__(kBlock) void k_tile_start(TileArgs a, uint32_t* __restrict__ ranges, int64_t words,
                                                       int64_t groups, uint4* __restrict__ sample) {
  __shared__ RectLds s_rect;
  __shared__ uint32_t s_sum[kWaves], s_box[kWaves];
  for (int64_t k = (int64_t)blockIdx.x * kBlock + threadIdx.x; k < words; k += (int64_t)gridDim.x * kBlock)
    ranges[k] = 0u;
  if (blockIdx.x >= (unsigned)kSampleGroups) return;
  // groups of kPer records over all views; a group of the sample may straddle two views, which only the estimate sees
  const int64_t i = groups * blockIdx.x / kSampleGroups * kPer + threadIdx.x;
  const int4 b = i < a.n ? a.bin[i] : make_int4(0, 0, 0, 0);
  const TileRect r = block_rect(s_rect, b, 1 << 12, 1 << 12);
  const uint32_t sum = wave_scan_u32(b.w > 0 ? (uint32_t)b.w : 0u);
  const uint32_t box = wave_top_u32(b.w > 0 ? (uint32_t)b.w : 0u);
  if ((threadIdx.x & (kWave - 1)) == kWave - 1) {
    s_sum[threadIdx.x / kWave] = sum;
    s_box[threadIdx.x / kWave] = box;
  }
  __syncthreads();
  if (threadIdx.x == 0)
    sample[blockIdx.x] = make_uint4((uint32_t)(r.w * r.h), s_sum[0] + s_sum[1] + s_sum[2] + s_sum[3],
                                    max(max(s_box[0], s_box[1]), max(s_box[2], s_box[3])), 0u);
}
// Whether the pairs are worth counting by tile (the same in every workgroup).
__device__ __forceinline__ bool worth_it(const uint4* __restrict__ sample) {
  static_assert(kSampleGroups == kWave, "one sample per lane");
  const uint4 x = sample[lane_id()];
  const uint32_t most = wave_top_u32(x.y);
  if (most > kMostGroupPairs && most > (uint64_t)kMostBoxes * wave_top_u32(x.z)) return false;
  // (64 rectangles of at most 2^24 tiles fit 32 bits, 64 times 2^27 pairs do not)
  const uint64_t pairs = ((uint64_t)last_lane(wave_scan_u32(x.y >> 16)) << 16) + last_lane(wave_scan_u32(x.y & 0xffffu));
  return 2 * (uint64_t)last_lane(wave_scan_u32(x.x)) <= kTilesPerTwoPairs * pairs;
}

// ---------------------------------------------------------------------------
// 1. count
// ---------------------------------------------------------------------------
// A tile's count gets one global add per workgroup that meets the tile:
// same-address atomics take turns (about 11 ns each), and one per pair took as
// long as the sort on the longest lists.
template <bool CULL>
__global__ __launch_bounds__(kBlock) void k_tile_count(TileArgs a, uint2* __restrict__ ranges, TileWs ws, ViewSet vs) {
  extern __shared__ uint32_t s_tab[];
  __shared__ WalkLds<CULL> s_walk[kWaves];
  __shared__ RectLds s_rect;
  __shared__ uint32_t s_sum[kWaves];
  __shared__ uint32_t s_st[3][kWaves];
  const int v = blockIdx.y;
  const int64_t i = record_of((int64_t)blockIdx.x * kPer);
  const int4 b = load_record(a, v, i);
  const int32_t tiles_x = vs.v[v].tiles_x;
  const TileRect r = block_rect(s_rect, b, tiles_x, vs.v[v].tiles_y);
  const int32_t fit = r.w > 0 ? a.table / r.w : 1;
  const int32_t height = worth_it(ws.sample) ? r.h : 0;
  for (int32_t y = 0; y < height; y += fit) {
    const int32_t rows = r.h - y < fit ? r.h - y : fit, cells = rows * r.w;
    __syncthreads();  // the previous band's table is read
    for (int32_t t = threadIdx.x; t < cells; t += kBlock) s_tab[t] = 0u;
    __syncthreads();
    walk_rows<CULL>(s_walk[threadIdx.x / kWave], a, v, i, b, r, r.y0 + y, rows,
                    [&](int32_t t, uint32_t, uint32_t) { atomicAdd(&s_tab[t], 1u); });
    __syncthreads();
    uint2* out = ranges + vs.v[v].tile_base + (r.y0 + y) * tiles_x + r.x0;
    for (int32_t t = threadIdx.x; t < cells; t += kBlock) {
      const uint32_t c = s_tab[t];
      const int32_t row = t / r.w;
      if (c) atomicAdd(&out[row * tiles_x + (t - row * r.w)].y, c);
    }
  }
  const bool drawn = b.w > 0;
  const uint32_t sum = drawn ? (uint32_t)b.w : 0u, vis = drawn ? 1u : 0u;  // 64 boxes of at most 2^19 tiles: 32 bits
  uint32_t nzmin = drawn ? ~(uint32_t)b.z : 0u, zmax = drawn ? (uint32_t)b.z : 0u;
  const uint32_t wsum = wave_scan_u32(sum), wvis = wave_scan_u32(vis);
  nzmin = wave_top_u32(nzmin);
  zmax = wave_top_u32(zmax);
  const int w = threadIdx.x / kWave;
  if ((threadIdx.x & (kWave - 1)) == kWave - 1) {
    s_sum[w] = wsum;
    s_st[0][w] = nzmin;
    s_st[1][w] = zmax;
    s_st[2][w] = wvis;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t total = 0, lo = 0u, hi = 0u, seen = 0u;
    for (int k = 0; k < kWaves; ++k) {
      total += s_sum[k];
      lo = s_st[0][k] > lo ? s_st[0][k] : lo;
      hi = s_st[1][k] > hi ? s_st[1][k] : hi;
      seen += s_st[2][k];
    }
    const int64_t g = (int64_t)v * gridDim.x + blockIdx.x;
    ws.sum[g] = total;  // kPer boxes of at most 2^19 tiles
    ws.zmin[g] = ~lo;
    ws.zmax[g] = hi;
    ws.vis[g] = seen;
  }
}

// ---------------------------------------------------------------------------
// 2. scan
// ---------------------------------------------------------------------------
constexpr int kScanT = 1024;
constexpr int kScanW = kScanT / kWave;
constexpr int kScanPer = 8;  // values of a thread per round, kScanT apart

// Exclusive scan of a round's kScanT kScanPer values, value j of thread t at
// j kScanT + t; returns the round's total.  Two barriers; lds is used again
// only after another barrier of the caller's.
__device__ __forceinline__ uint32_t scan_round(uint32_t (&x)[kScanPer], uint32_t* lds /* kScanPer kScanW + 1 */) {
  const int w = threadIdx.x / kWave, lane = threadIdx.x & (kWave - 1);
  uint32_t inc[kScanPer];
#pragma unroll
  for (int j = 0; j < kScanPer; ++j) {
    inc[j] = wave_scan_u32(x[j]);
    if (lane == kWave - 1) lds[j * kScanW + w] = inc[j];
  }
  __syncthreads();
  if (w == 0) {
    static_assert(kScanPer * kScanW == 2 * kWave, "two wave totals per lane");
    const uint32_t a = lds[2 * lane], b = lds[2 * lane + 1];
    const uint32_t s = wave_scan_u32(a + b);
    lds[2 * lane] = s - a - b;
    lds[2 * lane + 1] = s - b;
    if (lane == kWave - 1) lds[2 * kWave] = s;
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kScanPer; ++j) x[j] = lds[j * kScanW + w] + inc[j] - x[j];
  return lds[2 * kWave];
}
__device__ __forceinline__ uint32_t length_bucket(uint32_t c) { return c == 0 ? 32u : (uint32_t)__clz((int)c); }
// Lanes of the wave with the same bucket (6 bits: 0..32, and 63 for no tile).
__device__ __forceinline__ uint64_t bucket_lanes(uint32_t b) {
  uint64_t m = ~0ull;
#pragma unroll
  for (int bit = 0; bit < 6; ++bit) {
    const uint64_t bb = __builtin_amdgcn_ballot_w64(((b >> bit) & 1u) != 0u);
    m &= ((b >> bit) & 1u) ? bb : ~bb;
  }
  return m;
}

// Workgroup 0: counts (ranges[t].y) -> [start, start) per tile ([0, 0) if
// empty; k_tile_place moves the ends), the sort slices of long lists, the
// tiles' length buckets and their counts per kOrderTiles tiles (for the
// processing order), the longest list.  Workgroup 1: the counting workgroups'
// pair totals turned into starts, and the statistics.  One workgroup reads
// little more than a cache line per clock, so its loads are coalesced (eight
// consecutive values per thread took 28 us for 8,160 tiles and 11,700 totals,
// this 11 us).
__global__ __launch_bounds__(kScanT) void k_tile_scan(uint2* __restrict__ ranges, int32_t tiles, int64_t nb, TileWs ws,
                                                      uint64_t* __restrict__ host) {
  const int w = threadIdx.x / kWave, lane = threadIdx.x & (kWave - 1);
  __shared__ uint32_t lds[2][2][kScanPer * kScanW + 1];
  int side = 0;
  if (blockIdx.x == 0) {
    constexpr int kGroups = kScanT * kScanPer / kOrderTiles, kPerGroup = kScanPer / kGroups;
    __shared__ uint32_t s_hist[2][kGroups][kLengthBuckets];
    __shared__ uint32_t s_top[kScanW];
    for (int k = threadIdx.x; k < 2 * kGroups * kLengthBuckets; k += kScanT) (&s_hist[0][0][0])[k] = 0u;
    __shared__ uint64_t s_all[kScanW];
    uint32_t pairs = 0, slices = 0, longest = 0;
    uint64_t mine = 0;  // in 64 bits, as the boxes' total
    for (int32_t c0 = 0; c0 < tiles; c0 += kScanT * kScanPer, side ^= 1) {
      const int32_t t0 = c0 + (int32_t)threadIdx.x;
      uint32_t c[kScanPer], at[kScanPer], sl[kScanPer];
      // clamped, so that no branch keeps the loads from being in flight together
#pragma unroll
      for (int j = 0; j < kScanPer; ++j) c[j] = ranges[t0 + j * kScanT < tiles ? t0 + j * kScanT : tiles - 1].y;
      __syncthreads();  // s_hist of this side is clear
      uint32_t some = 0;
#pragma unroll
      for (int j = 0; j < kScanPer; ++j) {
        const int32_t t = t0 + j * kScanT;
        c[j] = t < tiles ? c[j] : 0u;
        longest = c[j] > longest ? c[j] : longest;
        mine += c[j];
        at[j] = c[j];
        sl[j] = slices_of(c[j]);
        some |= sl[j];
        const uint32_t b = t < tiles ? length_bucket(c[j]) : 63u;
        const uint64_t m = bucket_lanes(b);
        if (b != 63u) {
          if (lanes_below(m) == 0u) atomicAdd(&s_hist[side][j / kPerGroup][b], (uint32_t)__popcll(m));
          ws.bucket[t] = (uint8_t)b;
        }
      }
      const uint32_t all = scan_round(at, lds[side][0]);
#pragma unroll
      for (int j = 0; j < kScanPer; ++j) {
        const int32_t t = t0 + j * kScanT;
        const uint32_t s = pairs + at[j];
        if (t < tiles) ranges[t] = c[j] ? make_uint2(s, s) : make_uint2(0u, 0u);
      }
      pairs += all;
      if (__syncthreads_or(some != 0u)) {
        const uint32_t more = scan_round(sl, lds[side][1]);
#pragma unroll
        for (int j = 0; j < kScanPer; ++j) {
          uint32_t q = slices + sl[j];
          for (uint32_t k = 0; k < slices_of(c[j]); ++k, ++q)
            if (q < (uint32_t)kMaxSlices) ws.slices[q] = make_uint2((uint32_t)(t0 + j * kScanT), k);
        }
        slices += more;
      }
      // the adds to s_hist came before the scan's barriers
      if (threadIdx.x < kGroups * kLengthBuckets) {
        const int g = threadIdx.x / kLengthBuckets, b = threadIdx.x % kLengthBuckets;
        if (c0 + g * kOrderTiles < tiles) ws.hist[(c0 / kOrderTiles + g) * kLengthBuckets + b] = s_hist[side][g][b];
        s_hist[side][g][b] = 0u;
      }
    }
    longest = wave_top_u32(longest);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) mine += __shfl_xor(mine, o, kWave);
    if (lane == 0) { s_top[w] = longest; s_all[w] = mine; }
    __syncthreads();
    if (threadIdx.x == 0) {
      for (int k = 1; k < kScanW; ++k) {
        longest = s_top[k] > longest ? s_top[k] : longest;
        mine += s_all[k];
      }
      ws.stats[4] = host[4] = longest;
      ws.stats[5] = host[5] = slices;
      ws.stats[6] = host[6] = mine;
    }
    return;
  }
  __shared__ uint32_t s_red[2][kScanW];
  __shared__ uint64_t s_sum[2][kScanW];
  uint64_t total = 0, vis = 0;  // in 64 bits: 2^30 pairs or more have to be told from fewer
  uint32_t run = 0, nzmin = 0u, zmax = 0u;  // nzmin: ~zmin
  for (int64_t k0 = 0; k0 < nb; k0 += kScanT * kScanPer, side ^= 1) {
    const int64_t k = k0 + (int64_t)threadIdx.x;
    uint32_t c[kScanPer], lo[kScanPer], hi[kScanPer], seen[kScanPer];
#pragma unroll
    for (int j = 0; j < kScanPer; ++j) {
      const int64_t q = k + j * kScanT < nb ? k + j * kScanT : nb - 1;
      c[j] = ws.sum[q];
      lo[j] = ws.zmin[q];
      hi[j] = ws.zmax[q];
      seen[j] = ws.vis[q];
    }
#pragma unroll
    for (int j = 0; j < kScanPer; ++j) {
      const bool in = k + j * kScanT < nb;
      c[j] = in ? c[j] : 0u;
      total += c[j];
      vis += in ? seen[j] : 0u;
      nzmin = ~lo[j] > nzmin ? ~lo[j] : nzmin;  // past the end: the last one again
      zmax = hi[j] > zmax ? hi[j] : zmax;
    }
    const uint32_t all = scan_round(c, lds[side][0]);
#pragma unroll
    for (int j = 0; j < kScanPer; ++j)
      if (k + j * kScanT < nb) ws.sum[k + j * kScanT] = run + c[j];
    run += all;
  }
  nzmin = wave_top_u32(nzmin);
  zmax = wave_top_u32(zmax);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    vis += __shfl_xor(vis, o, kWave);
    total += __shfl_xor(total, o, kWave);
  }
  if (lane == 0) { s_red[0][w] = nzmin; s_red[1][w] = zmax; s_sum[0][w] = vis; s_sum[1][w] = total; }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int k = 1; k < kScanW; ++k) {
      nzmin = s_red[0][k] > nzmin ? s_red[0][k] : nzmin;
      zmax = s_red[1][k] > zmax ? s_red[1][k] : zmax;
      vis += s_sum[0][k];
      total += s_sum[1][k];
    }
    const uint64_t out[4] = {total, vis, vis ? ~nzmin : 0u, zmax};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      ws.stats[k] = out[k];
      host[k] = out[k];
    }
  }
}

// ---------------------------------------------------------------------------
// 3. offsets and processing order
// ---------------------------------------------------------------------------
// The tile order of kOrderTiles tiles: position = tiles of longer buckets, plus
// the bucket's tiles in earlier groups (both from the groups' counts), plus
// the rank inside the group (per-wave counts, then ballots), so inside a
// bucket the tiles keep ascending id.
struct OrderLds {
  uint32_t next[kWaves][kLengthBuckets];  // a wave's count of a bucket, then its next position
  uint32_t tot[kLengthBuckets], before[kLengthBuckets];
  uint8_t bucket[kOrderTiles];
};
__device__ __forceinline__ void order_group(OrderLds& s, int32_t group, int32_t tiles,
                                            const uint8_t* __restrict__ bucket, const uint32_t* __restrict__ hist,
                                            uint32_t* __restrict__ order) {
  const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
  const int32_t groups = (tiles + kOrderTiles - 1) / kOrderTiles, t0 = group * kOrderTiles;
  const int32_t nt = tiles - t0 < kOrderTiles ? tiles - t0 : kOrderTiles;
  for (int k = threadIdx.x; k < kWaves * kLengthBuckets; k += kBlock) (&s.next[0][0])[k] = 0u;
  if (threadIdx.x < kLengthBuckets) {
    uint32_t all = 0, pre = 0;
#pragma unroll 8
    for (int32_t g = 0; g < groups; ++g) {
      const uint32_t h = hist[g * kLengthBuckets + threadIdx.x];
      all += h;
      pre += g < group ? h : 0u;
    }
    s.tot[threadIdx.x] = all;
    s.before[threadIdx.x] = pre;
  }
  for (int32_t t = threadIdx.x; t < nt; t += kBlock) s.bucket[t] = bucket[t0 + t];
  __syncthreads();
  const int32_t per = (nt + kBlock - 1) / kBlock * kWave;  // tiles of a wave
  for (int32_t t = w * per + lane; t < (w + 1) * per; t += kWave) {
    const uint32_t b = t < nt ? s.bucket[t] : 63u;
    const uint64_t m = bucket_lanes(b);
    if (b != 63u && lanes_below(m) == 0u) s.next[w][b] += (uint32_t)__popcll(m);
  }
  __syncthreads();
  if (threadIdx.x < kLengthBuckets) {
    uint32_t run = s.before[threadIdx.x];
    for (int k = 0; k < (int)threadIdx.x; ++k) run += s.tot[k];
    for (int k = 0; k < kWaves; ++k) {
      const uint32_t c = s.next[k][threadIdx.x];
      s.next[k][threadIdx.x] = run;
      run += c;
    }
  }
  __syncthreads();
  for (int32_t t = w * per + lane; t < (w + 1) * per; t += kWave) {
    const uint32_t b = t < nt ? s.bucket[t] : 63u;
    const uint64_t m = bucket_lanes(b);
    uint32_t pos = 0;
    if (b != 63u) pos = s.next[w][b] + lanes_below(m);
    if (b != 63u && pos < (uint32_t)tiles) order[pos] = (uint32_t)(t0 + t);
    wave_sync();  // the bucket's lanes have read the position before its first lane moves it
    if (b != 63u && lanes_below(m) == 0u) s.next[w][b] = pos + (uint32_t)__popcll(m);
    wave_sync();
  }
}

// Exclusive scan of tiles_touched over the records (the workgroups' starts
// come from k_tile_scan); after the views, one row of workgroups for the
// processing order.
constexpr int kOffsetItems = 4;  // groups of kPer records of a workgroup

__global__ __launch_bounds__(kBlock) void k_tile_offsets(const int4* __restrict__ bin, int64_t n, int32_t views,
                                                         int32_t tiles, TileWs ws,
                                                         uint32_t* __restrict__ offsets,
                                                         uint32_t* __restrict__ order) {
  __shared__ union Lds {
    uint32_t w[kOffsetItems][kWaves];
    OrderLds order;
  } s;
  if ((int32_t)blockIdx.y == views) {
    for (int32_t g = blockIdx.x; g * kOrderTiles < tiles; g += gridDim.x) {
      order_group(s.order, g, tiles, ws.bucket, ws.hist, order);
      __syncthreads();
    }
    return;
  }
  const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
  const int64_t view = (int64_t)blockIdx.y * n, first = (int64_t)blockIdx.x * (kOffsetItems * kPer);
  const int64_t groups = (n + kPer - 1) / kPer;
  uint32_t x[kOffsetItems], inc[kOffsetItems];
#pragma unroll
  for (int q = 0; q < kOffsetItems; ++q) {
    const int64_t i = first + q * kPer + threadIdx.x;
    const int32_t c = bin[view + (i < n ? i : n - 1)].w;
    x[q] = i < n && c > 0 ? (uint32_t)c : 0u;
  }
#pragma unroll
  for (int q = 0; q < kOffsetItems; ++q) {
    inc[q] = wave_scan_u32(x[q]);
    if (lane == kWave - 1) s.w[q][w] = inc[q];
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < kOffsetItems; ++q) {
    const int64_t i = first + q * kPer + threadIdx.x;
    if (i >= n) break;
    uint32_t at = ws.sum[(int64_t)blockIdx.y * groups + (int64_t)blockIdx.x * kOffsetItems + q];
#pragma unroll
    for (int k = 0; k < kWaves; ++k) at += k < w ? s.w[q][k] : 0u;
    offsets[view + i] = at + inc[q] - x[q];
  }
}

// ---------------------------------------------------------------------------
// 4. place
// ---------------------------------------------------------------------------
// Entry = (depth - zmin) << ibits | record of the view.  The workgroup counts
// its pairs per tile again, takes room in each tile's run with one add on the
// run's end (ranges[t].y, at its start before), and hands the room out in LDS.
template <bool CULL>
__global__ __launch_bounds__(kBlock) void k_tile_place(TileArgs a, uint2* __restrict__ ranges, uint32_t zmin,
                                                       int32_t ibits, int64_t pairs, uint64_t* __restrict__ entries,
                                                       uint32_t* __restrict__ flag, ViewSet vs) {
  extern __shared__ uint32_t s_tab[];
  __shared__ WalkLds<CULL> s_walk[kWaves];
  __shared__ RectLds s_rect;
  const int v = blockIdx.y;
  if (blockIdx.x == 0 && v == 0 && threadIdx.x == 0) *flag = 0u;
  const int64_t i = record_of((int64_t)blockIdx.x * kPer);
  const int4 b = load_record(a, v, i);
  const int32_t tiles_x = vs.v[v].tiles_x;
  const TileRect r = block_rect(s_rect, b, tiles_x, vs.v[v].tiles_y);
  const int32_t fit = r.w > 0 ? a.table / r.w : 1;
  for (int32_t y = 0; y < r.h; y += fit) {
    const int32_t rows = r.h - y < fit ? r.h - y : fit, cells = rows * r.w;
    __syncthreads();  // the previous band's table is used up
    for (int32_t t = threadIdx.x; t < cells; t += kBlock) s_tab[t] = 0u;
    __syncthreads();
    walk_rows<CULL>(s_walk[threadIdx.x / kWave], a, v, i, b, r, r.y0 + y, rows,
                    [&](int32_t t, uint32_t, uint32_t) { atomicAdd(&s_tab[t], 1u); });
    __syncthreads();
    uint2* out = ranges + vs.v[v].tile_base + (r.y0 + y) * tiles_x + r.x0;
    for (int32_t t = threadIdx.x; t < cells; t += kBlock) {
      const uint32_t c = s_tab[t];
      const int32_t row = t / r.w;
      if (c) s_tab[t] = atomicAdd(&out[row * tiles_x + (t - row * r.w)].y, c);
    }
    __syncthreads();
    walk_rows<CULL>(s_walk[threadIdx.x / kWave], a, v, i, b, r, r.y0 + y, rows,
                    [&](int32_t t, uint32_t z, uint32_t who) {
      const uint32_t at = atomicAdd(&s_tab[t], 1u);
      if ((int64_t)at < pairs) entries[at] = ((uint64_t)(z - zmin) << ibits) | (uint64_t)who;
    });
  }
}

// ---------------------------------------------------------------------------
// 5. sort
// ---------------------------------------------------------------------------
// Three sizes of workgroup, so that short lists do not hold the LDS of long
// ones: a kernel's latency (loads, a dozen barriers) is hidden by the
// workgroups a CU holds at once.
constexpr int kShortThreads = 128, kShortItems = 4;    // lists of up to 512 entries
constexpr int kMidThreads = 256, kMidItems = 8;        // up to 2,048
constexpr int kLongThreads = 1024, kLongItems = 8;     // longer ones, in slices of up to 8,192
static_assert(kShortThreads * kShortItems == kShortCap && kMidThreads * kMidItems == kMidCap &&
                  kLongThreads * kLongItems == kLongCap, "list classes");

template <int T, int ITEMS>
struct SortLds {
  static constexpr int cap = T * ITEMS;
  uint64_t key[cap];
  uint32_t cnt[cap];
  uint32_t red[2][T / kWave];
  uint32_t wsum[T / kWave];
  uint32_t fill;
};

// Bitonic sort of the first n keys in LDS (padded to a power of two).
template <int T, int ITEMS>
__device__ __forceinline__ void bitonic(SortLds<T, ITEMS>& s, uint32_t n) {
  uint32_t p = 2;
#pragma unroll 1
  while (p < n) p <<= 1;
  for (uint32_t i = n + threadIdx.x; i < p; i += T) s.key[i] = ~0ull;
  __syncthreads();
#pragma unroll 1
  for (uint32_t k = 2; k <= p; k <<= 1)
#pragma unroll 1
    for (uint32_t j = k >> 1; j > 0; j >>= 1) {
      for (uint32_t q = threadIdx.x; q < p / 2; q += T) {
        const uint32_t i = 2 * q - (q & (j - 1)), l = i + j;
        const uint64_t x = s.key[i], y = s.key[l];
        if ((x > y) == ((i & k) == 0)) {
          s.key[i] = y;
          s.key[l] = x;
        }
      }
      __syncthreads();
    }
}

struct ListOut {
  uint32_t* vals;
  uint64_t* keys;     // NULL, or (tile << 32) | depth bits
  uint64_t tile_key;  // tile << 32
  uint32_t vbase, zmin;
  int32_t ibits;
  uint64_t imask;
  __device__ __forceinline__ uint32_t depth(uint64_t key) const { return (uint32_t)(key >> ibits); }
  __device__ __forceinline__ void put(uint64_t at, uint64_t key) const {
    vals[at] = vbase + (uint32_t)(key & imask);
    if (keys) keys[at] = tile_key | (uint64_t)(depth(key) + zmin);
  }
};

// Exclusive scan, in place in s.cnt, of nb counts read from `from` (nb a
// multiple of T); returns whether a count is above kBucketMax.
constexpr uint32_t kBucketMax = 16;

template <int T, int ITEMS>
__device__ __forceinline__ bool scan_buckets(SortLds<T, ITEMS>& s, const uint32_t* from, uint32_t nb) {
  constexpr int W = T / kWave;
  const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
  const uint32_t per = nb / T;  // thread t owns `per` consecutive counts
  uint32_t c[ITEMS], sum = 0, most = 0;
#pragma unroll
  for (int q = 0; q < ITEMS; ++q) {
    c[q] = (uint32_t)q < per ? from[threadIdx.x * per + q] : 0u;
    sum += c[q];
    most = c[q] > most ? c[q] : most;
  }
  const uint32_t inc = wave_scan_u32(sum);
  if (lane == kWave - 1) s.wsum[w] = inc;
  const bool bunched = __syncthreads_or(most > kBucketMax) != 0;
  uint32_t run = inc - sum;
#pragma unroll
  for (int q = 0; q < W; ++q) run += q < w ? s.wsum[q] : 0u;
#pragma unroll
  for (int q = 0; q < ITEMS; ++q) {
    if ((uint32_t)q < per) s.cnt[threadIdx.x * per + q] = run;
    run += c[q];
  }
  __syncthreads();
  return bunched;
}

// Sorts n (1..cap) distinct keys, thread t holding keys t, t + T, ..., and
// writes them to list positions at + 0..n-1.  The keys are spread over buckets
// of equal depth width between the smallest and the largest depth (a power of
// two not below n, so one or two keys each where depths are even), placed
// bucket by bucket, and each key finds its place in its bucket by comparing
// with the bucket's other keys.  Lists of a scene of surfaces have most of
// their depths in a few narrow bands: where a bucket gets more than kBucketMax
// keys, each bucket of c keys is cut into c of equal width and the keys are
// spread again.  Where that is not enough either (equal depths) the run is
// sorted by a bitonic network, whose cost does not depend on the values.
template <int T, int ITEMS>
__device__ __forceinline__ void sort_run(SortLds<T, ITEMS>& s, const uint64_t (&key)[ITEMS], uint32_t n, uint64_t at,
                                         const ListOut& out) {
  constexpr int W = T / kWave;
  const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
  uint32_t nb = T;  // at least one bucket per thread
  while (nb < n) nb <<= 1;
  uint32_t nlo = 0u, hi = 0u;  // ~smallest, largest depth
#pragma unroll
  for (int k = 0; k < ITEMS; ++k) {
    if (k * T + threadIdx.x < n) {
      const uint32_t d = out.depth(key[k]);
      nlo = ~d > nlo ? ~d : nlo;
      hi = d > hi ? d : hi;
    }
  }
  nlo = wave_top_u32(nlo);
  hi = wave_top_u32(hi);
  if (lane == 0) { s.red[0][w] = nlo; s.red[1][w] = hi; }
  for (uint32_t b = threadIdx.x; b < nb; b += T) s.cnt[b] = 0u;
  __syncthreads();
#pragma unroll
  for (int k = 0; k < W; ++k) {
    nlo = s.red[0][k] > nlo ? s.red[0][k] : nlo;
    hi = s.red[1][k] > hi ? s.red[1][k] : hi;
  }
  // d - lo and the product round monotonically, so buckets are in depth order
  const uint32_t lo = ~nlo;
  const float scale = (float)nb / ((float)(hi - lo) + 1.f);
  auto spread = [&](uint64_t k) { return (float)(out.depth(k) - lo) * scale; };
  uint32_t place[ITEMS];  // bucket | rank in it << 16
  static_assert(T * ITEMS <= 65536, "16 bits each");
#pragma unroll
  for (int k = 0; k < ITEMS; ++k) {
    place[k] = 0;
    if (k * T + threadIdx.x < n) {
      const uint32_t q = (uint32_t)spread(key[k]), b = q < nb ? q : nb - 1;
      place[k] = b | (atomicAdd(&s.cnt[b], 1u) << 16);
    }
  }
  __syncthreads();
  if (scan_buckets(s, s.cnt, nb)) {
    uint32_t* fine = reinterpret_cast<uint32_t*>(s.key);  // no key is stored yet
    for (uint32_t b = threadIdx.x; b < nb; b += T) fine[b] = 0u;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
      if (k * T + threadIdx.x < n) {
        const uint32_t b = place[k] & 0xffffu, b0 = s.cnt[b], b1 = b + 1 < nb ? s.cnt[b + 1] : n;
        const float x = spread(key[k]) - (float)b;  // [0, 1), or 1 and more in the last bucket
        const uint32_t q = b0 + (uint32_t)(x * (float)(b1 - b0)), f = q < b1 ? q : b1 - 1;
        place[k] = f | (atomicAdd(&fine[f], 1u) << 16);
      }
    }
    __syncthreads();
    if (scan_buckets(s, fine, nb)) {
#pragma unroll
      for (int k = 0; k < ITEMS; ++k) {
        const uint32_t i = k * T + threadIdx.x;
        if (i < n) s.key[i] = key[k];
      }
      bitonic(s, n);
      for (uint32_t i = threadIdx.x; i < n; i += T) out.put(at + i, s.key[i]);
      return;
    }
  }
#pragma unroll
  for (int k = 0; k < ITEMS; ++k)
    if (k * T + threadIdx.x < n) s.key[s.cnt[place[k] & 0xffffu] + (place[k] >> 16)] = key[k];
  __syncthreads();
#pragma unroll
  for (int k = 0; k < ITEMS; ++k) {
    if (k * T + threadIdx.x >= n) break;
    const uint32_t b = place[k] & 0xffffu, b0 = s.cnt[b], b1 = b + 1 < nb ? s.cnt[b + 1] : n;
    uint32_t less = 0;
    for (uint32_t j = b0; j < b1; ++j) less += s.key[j] < key[k] ? 1u : 0u;
    out.put(at + b0 + less, key[k]);
  }
}

__device__ __forceinline__ ListOut list_out(int32_t tile, const ViewSet& vs, int64_t n, uint32_t zmin, int32_t ibits,
                                            uint32_t* vals, uint64_t* keys) {
  ListOut out;
  out.vals = vals;
  out.keys = keys;
  out.tile_key = (uint64_t)(uint32_t)tile << 32;
  out.vbase = (uint32_t)((int64_t)view_of_tile(vs, tile) * n);
  out.zmin = zmin;
  out.ibits = ibits;
  out.imask = (1ull << ibits) - 1ull;
  return out;
}

// Lists of least + 1 .. T ITEMS entries, one workgroup per tile (the others
// exit).  No list reaches past `pairs`, the entries there is room for, whatever
// happened to the records between the counting and the placing.
__device__ __forceinline__ uint2 clamped(uint2 range, uint32_t pairs) {
  range.y = range.y < pairs ? range.y : pairs;
  range.x = range.x < range.y ? range.x : range.y;
  return range;
}
template <int T, int ITEMS>
__global__ __launch_bounds__(T) void k_tile_sort(const uint64_t* __restrict__ entries, uint2* ranges, uint32_t pairs,
                                                 uint32_t least, uint32_t zmin, int32_t ibits, int64_t n,
                                                 uint32_t* __restrict__ vals, uint64_t* __restrict__ keys,
                                                 ViewSet vs) {
  __shared__ SortLds<T, ITEMS> s;
  const int32_t tile = (int32_t)blockIdx.x;
  const uint2 given = ranges[tile], range = clamped(given, pairs);
  const uint32_t len = range.y - range.x;
  // (the last kernel of the lists is the one that takes all short ones)
  if (least == 0u && given.y > pairs && threadIdx.x == 0) ranges[tile] = range;
  if (len <= least || len > (uint32_t)(T * ITEMS)) return;
  const ListOut out = list_out(tile, vs, n, zmin, ibits, vals, keys);
  const uint64_t* run = entries + range.x;
  uint64_t key[ITEMS];
#pragma unroll
  for (int k = 0; k < ITEMS; ++k) {
    const uint32_t i = k * T + threadIdx.x;
    key[k] = i < len ? run[i] : 0ull;
  }
  sort_run(s, key, len, range.x, out);
}

// Keys of the run in [lo, hi) into LDS (the first cap of them); returns how
// many there are, and how many keys are below lo.
template <int T, int ITEMS>
__device__ __forceinline__ uint32_t gather_slice(SortLds<T, ITEMS>& s, const uint64_t* __restrict__ run, uint32_t len,
                                                 uint64_t lo, uint64_t hi, uint32_t* below) {
  constexpr int kAhead = 4;
  if (threadIdx.x == 0) s.fill = 0u;
  __syncthreads();
  uint32_t less = 0;
  for (uint32_t i0 = 0; i0 < len; i0 += kAhead * T) {
    uint64_t k[kAhead];
#pragma unroll
    for (int q = 0; q < kAhead; ++q) {
      const uint32_t i = i0 + q * T + threadIdx.x;
      k[q] = i < len ? run[i] : ~0ull;  // no key is ~0
    }
#pragma unroll
    for (int q = 0; q < kAhead; ++q) {
      less += k[q] < lo ? 1u : 0u;
      const bool in = k[q] >= lo && k[q] < hi;
      const uint64_t m = __builtin_amdgcn_ballot_w64(in);
      uint32_t first = 0;
      if (m != 0 && lane_id() == 0) first = atomicAdd(&s.fill, (uint32_t)__popcll(m));
      first = uniform_u32(first);
      const uint32_t at = first + lanes_below(m);
      if (in && at < (uint32_t)(T * ITEMS)) s.key[at] = k[q];
    }
  }
  less = last_lane(wave_scan_u32(less));
  if (lane_id() == 0) s.wsum[threadIdx.x / kWave] = less;
  __syncthreads();
  less = 0;
#pragma unroll
  for (int q = 0; q < T / kWave; ++q) less += s.wsum[q];
  const uint32_t count = s.fill;
  __syncthreads();
  *below = less;
  return count;
}

// Lists of more than kMidCap entries, one workgroup per slice (a list of up to
// kLongCap entries is one slice).  Longer lists are cut by depth into slices
// of about kSliceKeys: every workgroup of the list sorts the same sample of it,
// takes its slice's two bounds from there, and gathers the slice from the
// whole run, which is read once per slice, from L2.
__global__ __launch_bounds__(kLongThreads) void k_tile_sort_long(const uint64_t* __restrict__ entries,
                                                                 const uint2* __restrict__ ranges, uint32_t pairs,
                                                                 const uint2* __restrict__ slices, uint32_t zmin,
                                                                 int32_t ibits, int64_t n,
                                                                 uint32_t* __restrict__ vals,
                                                                 uint64_t* __restrict__ keys, ViewSet vs) {
  constexpr int T = kLongThreads, ITEMS = kLongItems;
  __shared__ SortLds<T, ITEMS> s;
  const uint2 item = slices[blockIdx.x];
  const int32_t tile = (int32_t)item.x;
  const uint32_t slice = item.y;
  const uint2 range = clamped(ranges[tile], pairs);
  const uint32_t len = range.y - range.x;
  const ListOut out = list_out(tile, vs, n, zmin, ibits, vals, keys);
  const uint64_t* run = entries + range.x;
  const uint32_t count_slices = slices_of(len);
  if (slice >= count_slices) return;
  uint64_t lo = 0ull, end = ~0ull;
  if (count_slices > 1) {
    // bounds of this slice: quantiles of kSample evenly spaced entries of the run
    for (uint32_t i = threadIdx.x; i < (uint32_t)kSample; i += T)
      s.key[i] = run[(uint32_t)(((uint64_t)i * len + len / 2) / kSample)];
    bitonic(s, kSample);
    if (slice > 0) lo = s.key[slice * (uint32_t)kSample / count_slices];
    if (slice + 1 < count_slices) end = s.key[(slice + 1) * (uint32_t)kSample / count_slices];
    __syncthreads();
  }
  // one turn, unless a slice came out too large: it is halved until it fits
  while (lo < end) {
    uint64_t hi = end;
    uint32_t below = 0, count = len;
    uint64_t key[ITEMS];
    if (count_slices > 1) {
      count = gather_slice(s, run, len, lo, hi, &below);
      while (count > (uint32_t)kLongCap) {
        hi = lo + (hi - lo) / 2;
        count = gather_slice(s, run, len, lo, hi, &below);
      }
#pragma unroll
      for (int k = 0; k < ITEMS; ++k) {
        const uint32_t i = k * T + threadIdx.x;
        key[k] = i < count ? s.key[i] : 0ull;
      }
    } else {
      uint32_t tid = threadIdx.x;
      asm volatile("" : "+v"(tid));  // keeps the eight addresses out of the registers around the loop
#pragma unroll
      for (int k = 0; k < ITEMS; ++k) {
        const uint32_t i = k * T + tid;
        key[k] = i < count ? run[i] : 0ull;
      }
    }
    __syncthreads();
    if (count > 0) sort_run(s, key, count, (uint64_t)range.x + below, out);
    __syncthreads();
    lo = hi;
  }
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
namespace {

int64_t max_blocks(int64_t nrec) { return nrec / kPer + 1 + GS_MAX_VIEWS; }

struct Grid {
  dim3 dim;
  size_t lds;
  TileArgs a;
  bool cull;
};
Grid tile_grid(const gs_projected_t* proj, const ViewSet& vs, int32_t V, int64_t n) {
  int32_t most = 1;
  for (int32_t v = 0; v < V; ++v) {
    const int32_t t = vs.v[v].tiles_x * vs.v[v].tiles_y;
    most = t > most ? t : most;
  }
  Grid g;
  g.a.bin = reinterpret_cast<const int4*>(proj->bin);
  g.a.rec = proj->rec;
  g.a.tile_cull = proj->tile_cull_log2_alpha;
  g.a.n = n;
  g.a.table = most < kTableTiles ? most : kTableTiles;
  g.lds = (size_t)g.a.table * 4;
  g.dim = dim3((unsigned)((n + kPer - 1) / kPer), (unsigned)V);
  g.cull = proj->tile_cull_log2_alpha < 0.f;
  return g;
}

}  // namespace

size_t tile_ws_bytes(int64_t nrec) {
  const int64_t nb = max_blocks(nrec);
  return 4 * align256(nb * 4) + align256(kTileStats * 8) +
         align256((size_t)kMaxOrderGroups * kLengthBuckets * 4) + align256((size_t)kMaxSlices * 8) +
         align256((size_t)kMaxOrderGroups * kOrderTiles) + align256((size_t)kSampleGroups * 16);
}

TileWs carve_tiles(void* ws, int64_t nrec) {
  const int64_t nb = max_blocks(nrec);
  char* p = static_cast<char*>(ws);
  TileWs t;
  t.sum = reinterpret_cast<uint32_t*>(p); p += align256(nb * 4);
  t.zmin = reinterpret_cast<uint32_t*>(p); p += align256(nb * 4);
  t.zmax = reinterpret_cast<uint32_t*>(p); p += align256(nb * 4);
  t.vis = reinterpret_cast<uint32_t*>(p); p += align256(nb * 4);
  t.stats = reinterpret_cast<uint64_t*>(p); p += align256(kTileStats * 8);
  t.hist = reinterpret_cast<uint32_t*>(p); p += align256((size_t)kMaxOrderGroups * kLengthBuckets * 4);
  t.slices = reinterpret_cast<uint2*>(p); p += align256((size_t)kMaxSlices * 8);
  t.bucket = reinterpret_cast<uint8_t*>(p); p += align256((size_t)kMaxOrderGroups * kOrderTiles);
  t.sample = reinterpret_cast<uint4*>(p);
  return t;
}

// Whether the counting by tile can run at all: the processing order's groups
// have to fit the workspace, a row of tiles the table.
bool tiles_eligible(const ViewSet& vs) {
  for (int32_t v = 0; v < vs.count; ++v)
    if (vs.v[v].tiles_x > kTableTiles) return false;
  return vs.tiles_total <= kMaxOrderGroups * kOrderTiles;
}

int32_t count_by_tile(const gs_projected_t* proj, const ViewSet& vs, int32_t V, int64_t n, uint32_t* ranges,
                      const TileWs& ws, uint64_t* host, hipStream_t s) {
  const Grid g = tile_grid(proj, vs, V, n);
  uint2* r2 = reinterpret_cast<uint2*>(ranges);
  const int64_t words = 2 * (int64_t)vs.tiles_total, nrec = (int64_t)V * n;
  TileArgs all = g.a;  // the records of all views
  all.n = nrec;
  const int64_t fill = (words + 4 * kBlock - 1) / (4 * kBlock);
  hipLaunchKernelGGL(k_tile_start, dim3((unsigned)(fill > kSampleGroups ? fill : kSampleGroups)), dim3(kBlock), 0, s,
                     all, ranges, words, (nrec + kPer - 1) / kPer, ws.sample);
  if (g.cull)
    hipLaunchKernelGGL(k_tile_count<true>, g.dim, dim3(kBlock), g.lds, s, g.a, r2, ws, vs);
  else
    hipLaunchKernelGGL(k_tile_count<false>, g.dim, dim3(kBlock), g.lds, s, g.a, r2, ws, vs);
  hipLaunchKernelGGL(k_tile_scan, dim3(2), dim3(kScanT), 0, s, r2, vs.tiles_total, (int64_t)g.dim.x * g.dim.y, ws,
                     host);
  MS_CHECK_LAUNCH("tile count");
  return GS_OK;
}

int32_t offsets_by_tile(const gs_projected_t* proj, const ViewSet& vs, int32_t V, int64_t n, const TileWs& ws,
                        uint32_t* offsets, uint32_t* tile_order, hipStream_t s) {
  constexpr int64_t per = kOffsetItems * kPer;
  hipLaunchKernelGGL(k_tile_offsets, dim3((unsigned)((n + per - 1) / per), (unsigned)V + 1), dim3(kBlock), 0, s,
                     reinterpret_cast<const int4*>(proj->bin), n, V, vs.tiles_total, ws, offsets, tile_order);
  MS_CHECK_LAUNCH("tile offsets");
  return GS_OK;
}

// Whether the lists are sorted by tile (max_list is 0 where the pairs were not
// counted by tile, or came out other than the records say).  Every slice of a long list reads the
// whole list, so the cost of one list grows with its square.
bool lists_by_tile_pay(const gs_bin_stats_t* stats) {
  return stats->max_list > 0 && stats->max_list <= kTileMaxList && stats->list_slices <= kMaxSlices;
}

int32_t lists_by_tile(const gs_projected_t* proj, const ViewSet& vs, int32_t V, int64_t n,
                      const gs_bin_stats_t* stats, const TileWs& ws, uint32_t* ranges, uint64_t* keys, uint32_t* vals,
                      void* sort_ws, hipStream_t s) {
  uint32_t* flag = static_cast<uint32_t*>(sort_ws);
  uint64_t* entries = reinterpret_cast<uint64_t*>(static_cast<char*>(sort_ws) + kSortHeaderBytes);
  uint2* r2 = reinterpret_cast<uint2*>(ranges);
  const int32_t tiles = vs.tiles_total;
  const uint32_t zmin = stats->zbits_min;
  int32_t ibits = 1;
  while (ibits < 31 && (int64_t(1) << ibits) < n) ++ibits;
  const Grid g = tile_grid(proj, vs, V, n);
  if (g.cull)
    hipLaunchKernelGGL(k_tile_place<true>, g.dim, dim3(kBlock), g.lds, s, g.a, r2, zmin, ibits, stats->n_isect,
                       entries, flag, vs);
  else
    hipLaunchKernelGGL(k_tile_place<false>, g.dim, dim3(kBlock), g.lds, s, g.a, r2, zmin, ibits, stats->n_isect,
                       entries, flag, vs);
  const uint32_t pairs = (uint32_t)stats->n_isect;
  // the longest lists first: they take longest
  if (stats->list_slices > 0)
    hipLaunchKernelGGL(k_tile_sort_long, dim3((unsigned)stats->list_slices), dim3(kLongThreads), 0, s, entries, r2,
                       pairs, ws.slices, zmin, ibits, n, vals, keys, vs);
  if (stats->max_list > kShortCap)
    hipLaunchKernelGGL((k_tile_sort<kMidThreads, kMidItems>), dim3((unsigned)tiles), dim3(kMidThreads), 0, s, entries,
                       r2, pairs, (uint32_t)kShortCap, zmin, ibits, n, vals, keys, vs);
  hipLaunchKernelGGL((k_tile_sort<kShortThreads, kShortItems>), dim3((unsigned)tiles), dim3(kShortThreads), 0, s,
                     entries, r2, pairs, 0u, zmin, ibits, n, vals, keys, vs);
  MS_CHECK_LAUNCH("tile lists");
  return GS_OK;
}

}  // namespace msplat
