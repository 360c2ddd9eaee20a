// a5-a7: per-tile compositing (Eq. (1)), argmax index and depth (Eq. (2),
// Sec. 4.1), importance / max-weight / area accumulation (Sec. 3.2, Eq. (3),
// Sec. 5.1), and the reverse-order backward restricted to an active mask
// (Sec. 5.2).
//
// Work mapping: a 256-thread workgroup per 16x16 tile (or per 8x8 quarter of
// a heavy tile, see work_item), one wave per 8x8 quarter, and inside a wave
// four 4x4 pixel groups, one per 16-lane row.  Per round the workgroup stages
// up to 256 consecutive list entries (record index, pixel box and the 48 or
// 64 bytes of the record the pass reads) in LDS with one gather per thread,
// while the next round's records and the list indices of the round after are
// already in flight.  Each thread then tests the entry it staged against the
// bounding rectangle of the still-active pixels of every group of the
// workgroup (pixel box, then an exact conservative ellipse-rectangle test); the
// ballots, expanded by each wave for its own groups, give every group its own
// stream of entries that can reach it (LDS offsets), and each group walks its
// stream in list order reading records with broadcast LDS loads.  Culled
// entries never reach alpha_min at those pixels, so culling never changes a
// result.  Groups whose pixels have all stopped drop the rest of their stream,
// and a wave ends when all its groups have.
#include <cmath>
#include <type_traits>

#include "common.hpp"

namespace msplat {

struct FwdOut {
  float* color;
  float* depth;
  int32_t* imax;
  float* t_final;
  uint32_t* last;
  uint32_t* n_contrib;
  uint8_t* hit;
  float* imp;
  float* wmax;
  uint32_t* area;
};

// Mid-point of the ray's intersections with the 1-sigma ellipsoid (Sec. 4.1),
// in the ellipsoid's scaled frame: t* = -(o'.d') / (d'.d'); d has unit camera
// z, so t* is a camera depth.  Double precision: it runs once per pixel.
// The camera travels by value: handing a reference into the kernel-argument
// view table to a call would make the compiler copy the whole table to
// per-thread scratch.
struct RayCam {
  float R[9];
  float t[3];
  float fx, fy, cx, cy;
};

struct MidDepth {
  float depth;
  uint32_t hit;
};

__device__ __noinline__ MidDepth mid_depth(const RayCam cam, const float* __restrict__ means,
                                           const float* __restrict__ scales, const float* __restrict__ quats,
                                           int64_t n, int64_t g, float pxc, float pyc) {
  double R[9];
  for (int k = 0; k < 9; ++k) R[k] = cam.R[k];
  const double c0 = -(R[0] * cam.t[0] + R[3] * cam.t[1] + R[6] * cam.t[2]);
  const double c1 = -(R[1] * cam.t[0] + R[4] * cam.t[1] + R[7] * cam.t[2]);
  const double c2 = -(R[2] * cam.t[0] + R[5] * cam.t[1] + R[8] * cam.t[2]);
  const double e0 = ((double)pxc - cam.cx) / cam.fx, e1 = ((double)pyc - cam.cy) / cam.fy;
  const double d0 = R[0] * e0 + R[3] * e1 + R[6];
  const double d1 = R[1] * e0 + R[4] * e1 + R[7];
  const double d2 = R[2] * e0 + R[5] * e1 + R[8];
  const double qw = quats[g], qx = quats[n + g], qy = quats[2 * n + g], qz = quats[3 * n + g];
  const double iq = 1.0 / sqrt(qw * qw + qx * qx + qy * qy + qz * qz);
  double w = qw * iq, x = qx * iq, y = qy * iq, z = qz * iq;
  double o0 = c0 - means[g], o1 = c1 - means[n + g], o2 = c2 - means[2 * n + g];
  double od = 0.0, dd = 0.0, oo = 0.0;
  // One axis of the ellipsoid (a column of its rotation) after the other: side
  // by side they take 72 registers, more than the kernels that call this.
  auto axis = [&](double q0, double q1, double q2, float scale) {
    const double is = 1.0 / (double)scale;
    const double ok = (q0 * o0 + q1 * o1 + q2 * o2) * is;
    const double dk = (q0 * d0 + q1 * d1 + q2 * d2) * is;
    od += ok * dk;
    dd += dk * dk;
    oo += ok * ok;
    asm volatile("" : "+v"(od), "+v"(dd), "+v"(oo), "+v"(w), "+v"(x), "+v"(y), "+v"(z));
  };
  axis(1.0 - 2.0 * (y * y + z * z), 2.0 * (x * y + w * z), 2.0 * (x * z - w * y), scales[g]);
  axis(2.0 * (x * y - w * z), 1.0 - 2.0 * (x * x + z * z), 2.0 * (y * z + w * x), scales[n + g]);
  axis(2.0 * (x * z + w * y), 2.0 * (y * z - w * x), 1.0 - 2.0 * (x * x + y * y), scales[2 * n + g]);
  MidDepth r;
  r.depth = (float)(-od / dd);
  r.hit = (od * od - dd * (oo - 1.0)) >= 0.0 ? 1u : 0u;
  return r;
}

// Value of another lane of the same 16-lane row (DPP control CTRL).
template <int CTRL>
__device__ __forceinline__ float dpp_take(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xF, 0xF, true));
}
// Sum and largest of two weights (>= 0) per lane over each 16-lane row, the
// first's in lanes 0-7 of a row, the second's in lanes 8-15 (the bank masks of
// the first adds keep one in either half, see row_sum9).  The accumulating
// forward then adds an entry's weights from one lane per group.
// Adding every lane's weight in LDS instead cost up to 240 cycles of the CU's
// LDS per entry (ds_add_f32 takes one lane at a time) and 60 for the maximum
// (lanes of one address take turns): three times the vector instructions of
// the walk.
struct SumMax {
  float sum, max;
};
__device__ __forceinline__ SumMax row_sum_max2(float w0, float w1) {
  SumMax r;
  asm("s_nop 1\n\t"
      "v_add_f32_dpp %0, %2, %2 row_ror:8 row_mask:0xf bank_mask:0x3\n\t"
      "v_max_f32_dpp %1, %2, %2 row_ror:8 row_mask:0xf bank_mask:0x3\n\t"
      "v_add_f32_dpp %0, %3, %3 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
      "v_max_f32_dpp %1, %3, %3 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
      "s_nop 0\n\t"
      "v_add_f32_dpp %0, %0, %0 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
      "v_max_f32_dpp %1, %1, %1 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
      "s_nop 0\n\t"
      "v_add_f32_dpp %0, %0, %0 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
      "v_max_f32_dpp %1, %1, %1 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
      "s_nop 0\n\t"
      "v_add_f32_dpp %0, %0, %0 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
      "v_max_f32_dpp %1, %1, %1 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf"
      : "=&v"(r.sum), "=&v"(r.max)
      : "v"(w0), "v"(w1));
  return r;
}
// Exchanges between the four 16-lane rows of one column (lanes j, 16 + j,
// 32 + j, 48 + j) with the gfx950 permlane swaps: permlane16_swap hands each
// row the values of the even and the odd row of its pair (rows 0-1, 2-3),
// permlane32_swap the values of the same row parity in the lower and upper
// pair.  Split work items use the rows as four consecutive entries of one
// pixel group's stream; the scans below combine them in row order.
struct RowsTwo {
  uint32_t a, b;
};
__device__ __forceinline__ RowsTwo rows_pair(uint32_t x) {
  const auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
  return {r[0], r[1]};
}
__device__ __forceinline__ RowsTwo rows_halves(uint32_t x) {
  const auto r = __builtin_amdgcn_permlane32_swap(x, x, false, false);
  return {r[0], r[1]};
}
struct RowScan {
  float incl, excl, total;
};
// Products over the rows of a column: inclusive and exclusive up to `row`,
// and over all four rows.
__device__ __forceinline__ RowScan rows_scan_mul(float x, int row) {
  const RowsTwo p = rows_pair(__float_as_uint(x));
  const float e = __uint_as_float(p.a), o = __uint_as_float(p.b);
  const float pair = e * o;
  const RowsTwo h = rows_halves(__float_as_uint(pair));
  const float lo = __uint_as_float(h.a), hi = __uint_as_float(h.b);
  const float in2 = (row & 1) ? pair : e, ex2 = (row & 1) ? e : 1.f;
  RowScan r;
  r.incl = row >= 2 ? lo * in2 : in2;
  r.excl = row >= 2 ? lo * ex2 : ex2;
  r.total = lo * hi;
  return r;
}
// Sums over the rows of a column: exclusive up to `row` and over all four.
__device__ __forceinline__ RowScan rows_scan_add(float x, int row) {
  const RowsTwo p = rows_pair(__float_as_uint(x));
  const float e = __uint_as_float(p.a), o = __uint_as_float(p.b);
  const float pair = e + o;
  const RowsTwo h = rows_halves(__float_as_uint(pair));
  const float lo = __uint_as_float(h.a), hi = __uint_as_float(h.b);
  const float ex2 = (row & 1) ? e : 0.f;
  RowScan r;
  r.incl = 0.f;
  r.excl = row >= 2 ? lo + ex2 : ex2;
  r.total = lo + hi;
  return r;
}
__device__ __forceinline__ float rows_sum(float x) {
  const RowsTwo p = rows_pair(__float_as_uint(x));
  const float pair = __uint_as_float(p.a) + __uint_as_float(p.b);
  const RowsTwo h = rows_halves(__float_as_uint(pair));
  return __uint_as_float(h.a) + __uint_as_float(h.b);
}
__device__ __forceinline__ uint32_t rows_sum_u32(uint32_t x) {
  const RowsTwo p = rows_pair(x);
  const RowsTwo h = rows_halves(p.a + p.b);
  return h.a + h.b;
}
__device__ __forceinline__ uint32_t rows_max_u32(uint32_t x) {
  const RowsTwo p = rows_pair(x);
  const uint32_t m = p.a > p.b ? p.a : p.b;
  const RowsTwo h = rows_halves(m);
  return h.a > h.b ? h.a : h.b;
}

__device__ __forceinline__ bool box_meets(int2 b, int32_t x0, int32_t x1, int32_t y0, int32_t y1) {
  // pixel box (lo | hi << 16) against the pixel rectangle [x0, x1] x [y0, y1]
  return (int32_t)((uint32_t)b.x >> 16) >= x0 && (b.x & 0xffff) <= x1 && (int32_t)((uint32_t)b.y >> 16) >= y0 &&
         (b.y & 0xffff) <= y1;
}

// One list entry as staged in LDS: record index, pixel box, the first 48
// bytes of its record (screen mean, scaled conic, colour and opacity) and,
// for blended depth, its camera depth.  Where there is no entry (past the list's
// end) or its index is corrupt (>= V n), the box is empty, so it is never drawn,
// and colour and depth are staged as zeros: a group walks to the longest of its
// wave's streams and multiplies what lies past its own by a weight of 0, which
// has to be finite, and row 0, read in its place, need not be (the projection
// leaves the rows of records that are not drawn unwritten).  The zeros are
// chosen when the entry is staged, a round after its loads: with the loads under
// the condition instead 3M Gaussians at 1920x1080 with accumulation took 603 us,
// so 556 (the backward takes the same either way).
struct Staged {
  __device__ __forceinline__ bool entry() const { return box.x != 0xffff; }
  uint32_t idx;
  int2 box;
  float4 r0, r1, r2;
  float z;
};
__device__ __forceinline__ Staged fetch_entry(const float* __restrict__ rec, const int32_t* __restrict__ bin,
                                              uint32_t r, bool in_list, int64_t nrec) {
  Staged e;
  const bool valid = in_list && (int64_t)r < nrec;
  r = valid ? r : 0u;
  e.idx = r;
  e.box = valid ? *reinterpret_cast<const int2*>(bin + 4 * (int64_t)r) : make_int2(0xffff, 0xffff);
  const float4* R4 = reinterpret_cast<const float4*>(rec + (int64_t)r * kRecFloats);
  e.r0 = R4[0];
  e.r1 = R4[1];
  e.r2 = R4[2];
  e.z = rec[(int64_t)r * kRecFloats + 12];
  return e;
}

struct Rect {
  int32_t x0, x1, y0, y1;
};

// Bounding rectangle of the set bits of a 16-lane group's mask (4x4 pixels,
// bit = 4 * row + column, non-zero) whose block starts at (gx0, gy0).
__device__ __forceinline__ Rect group_rect(uint32_t bits, int32_t gx0, int32_t gy0) {
  const uint32_t cols = (bits | (bits >> 4) | (bits >> 8) | (bits >> 12)) & 0xfu;
  Rect r;
  r.y0 = gy0 + ((int32_t)__builtin_ctz(bits) >> 2);
  r.y1 = gy0 + ((31 - (int32_t)__builtin_clz(bits)) >> 2);
  r.x0 = gx0 + (int32_t)__builtin_ctz(cols);
  r.x1 = gx0 + (31 - (int32_t)__builtin_clz(cols));
  return r;
}

// The same value, which the compiler does not know to be the same: what is
// computed from it is computed where it is used instead of being held in
// registers over the loops in between (registers set how many waves a SIMD
// holds in these kernels).
__device__ __forceinline__ int fresh(int x) {
  asm volatile("" : "+v"(x));
  return x;
}
__device__ __forceinline__ int32_t fresh_uniform(int32_t x) {
  asm volatile("" : "+s"(x));
  return x;
}
// One staged entry against the pixel centres of a group's rectangle: what
// ellipse_meets decides, for the many tests of a round.  `ox`, `oy`: the centre
// of the work item's first pixel minus the entry's mean; x0..y1: the
// rectangle, from that pixel.  A convex quadratic with its minimum outside a rectangle
// takes its least value there on one of the (at most two) edges that face the
// minimum, so two edges are tried instead of four: the one at the nearest x
// and the one at the nearest y (where the minimum lies between the edges, the
// nearest value is 0 and the point tried is one of the rectangle, so the
// result is never below the true minimum).  Same margin as ellipse_meets,
// far above the rounding of the approximate reciprocals.
struct EntryTest {
  float ox, oy, A, B, C, hiA, hiC, lim;
};
__device__ __forceinline__ EntryTest entry_test(float4 r0, float4 r1, int32_t ix0, int32_t iy0,
                                                float log2_alpha_min) {
  EntryTest t;
  t.ox = ((float)ix0 + 0.5f - r0.x) - r0.z;
  t.oy = ((float)iy0 + 0.5f - r0.y) - r0.w;
  t.A = r1.x;
  t.B = r1.y;
  t.C = r1.z;
  t.hiA = -0.5f * r1.y * __builtin_amdgcn_rcpf(r1.x);
  t.hiC = -0.5f * r1.y * __builtin_amdgcn_rcpf(r1.z);
  const float budget = r1.w - log2_alpha_min;
  t.lim = budget + 1e-3f * (1.f + fabsf(budget));
  return t;
}
__device__ __forceinline__ bool group_meets(const EntryTest& t, float x0, float x1, float y0, float y1) {
  const float lx = t.ox + x0, hx = t.ox + x1, ly = t.oy + y0, hy = t.oy + y1;
  const float nx = __builtin_amdgcn_fmed3f(0.f, lx, hx), ny = __builtin_amdgcn_fmed3f(0.f, ly, hy);
  const float yx = __builtin_amdgcn_fmed3f(t.hiC * nx, ly, hy), xy = __builtin_amdgcn_fmed3f(t.hiA * ny, lx, hx);
  const float qx = nx * (t.A * nx + t.B * yx) + t.C * yx * yx;
  const float qy = xy * (t.A * xy + t.B * ny) + t.C * ny * ny;
  return fminf(qx, qy) <= t.lim;
}

// List entries staged per workgroup round, at most one per thread.  A round
// costs its barriers and its streams whatever its length, so rounds are as long
// as LDS allows at six workgroups per CU (26,880 bytes each): the backward's
// double accumulators (72 bytes per entry) leave room for 192, its float ones
// and the forms without accumulators for 256.
constexpr int kFwdBatch = 256;
template <bool MASKED, bool DET>
constexpr int kBwdBatch = MASKED || DET ? 256 : 192;

// The groups' streams of one round.  Every thread tests its staged entry, still
// in registers, against all groups of the workgroup (four per wave, one per
// wave in a split work item), so an entry's test is set up once instead of
// once per wave, and the records need not be read back from LDS.  Wave c leaves
// the ballots of its 64 entries in mask[wave][group][c]; after the barrier each
// wave expands its own groups' masks into lists of entries.  Walking a list
// costs one LDS read per entry (two per read in the forward); walking the masks
// instead costs ten vector instructions per entry (two-word bit scans and
// clears per lane), and walking 64 entries at a time waits for the slowest of
// the four groups four times as often.
constexpr int kGroups = 4;
constexpr int kWaves = kBlock / kWave;
// The backward knows in which chunks a pixel still composites (PER_CHUNK), the
// forward only whether it does at the start of the round.
template <int BATCH, bool PER_CHUNK>
struct RoundLds {
  static constexpr int chunks = BATCH / kWave;
  uint64_t active[kWaves][PER_CHUNK ? chunks : 1];  // pixels of each wave that still composite
  uint64_t mask[kWaves][kGroups][chunks];
  __device__ __forceinline__ bool none_active() const {
    uint64_t any = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) any |= active[w][0];
    return uniform_u64(any) == 0;
  }
};
// `group_last` (or NULL): list positions from which on a group composites nothing.
// Returns the entries of this wave's chunk that some group walks.
template <int BATCH, bool PER_CHUNK>
__device__ __forceinline__ uint64_t test_round(RoundLds<BATCH, PER_CHUNK>& s, const uint32_t* group_last, uint32_t pos, bool split,
                                               int32_t ix0, int32_t iy0, int2 box, float4 r0, float4 r1, bool in,
                                               int wv, int lane, float log2_alpha_min) {
  if (wv >= RoundLds<BATCH, PER_CHUNK>::chunks) return 0;
  uint64_t any = 0;
  uint32_t lo = 0, hi = 0;  // lane 4 w + g keeps the mask of group g of wave w
  if (__builtin_amdgcn_ballot_w64(in) != 0) {
    const EntryTest t = entry_test(r0, r1, ix0, iy0, log2_alpha_min);
    uint32_t last = 0;
    if (group_last) last = group_last[lane & (kWaves * kGroups - 1)];
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      const uint64_t am = uniform_u64(s.active[w][PER_CHUNK ? wv : 0]);
#pragma unroll
      for (int g = 0; g < kGroups; ++g) {
        const uint32_t two = (uint32_t)(g < 2 ? am : am >> 32);
        const uint32_t bits = split && g > 0 ? 0u : (g & 1) ? two >> 16 : two & 0xffffu;
        if (bits == 0u) continue;
        const int32_t gx = split ? (w & 1) * 4 : (w & 1) * 8 + (g & 1) * 4;
        const int32_t gy = split ? (w >> 1) * 4 : (w >> 1) * 8 + (g >> 1) * 4;
        const Rect rg = group_rect(bits, gx, gy);
        bool rel = in && box_meets(box, ix0 + rg.x0, ix0 + rg.x1, iy0 + rg.y0, iy0 + rg.y1) &&
                   group_meets(t, (float)rg.x0, (float)rg.x1, (float)rg.y0, (float)rg.y1);
        if (group_last) rel = rel && pos < (uint32_t)__builtin_amdgcn_readlane((int)last, w * kGroups + g);
        const uint64_t m = __builtin_amdgcn_ballot_w64(rel);
        // (a vector instruction may read a scalar two instructions after another has written it)
        asm("s_nop 1\n\tv_writelane_b32 %0, %2, %4\n\tv_writelane_b32 %1, %3, %4"
            : "+v"(lo), "+v"(hi)
            : "s"((uint32_t)m), "s"((uint32_t)(m >> 32)), "n"(w * kGroups + g));
        any |= m;
      }
    }
  }
  if (lane < kWaves * kGroups)
    s.mask[lane / kGroups][lane & (kGroups - 1)][wv] = (uint64_t)lo | ((uint64_t)hi << 32);
  return any;
}
// Entries of this wave's groups, `unit` per staged entry; n[g]: their counts.
// By chunk, in a split work item: n[c] is where chunk c's part of the one
// group's stream ends (FILL: filled up with kNoEntry to a multiple of four).
// Without FILL (the backward, which reads no offset past a stream's end, but the
// first one of an empty stream) every stream begins with an offset in range,
// whatever the flush of the round before has left there.
constexpr uint16_t kNoEntry = 0xffff;
__device__ __forceinline__ int fill_four(uint16_t* stream, int n, int lane) {
  const int fill = -n & 3;
  if (lane < fill) stream[n + lane] = kNoEntry;
  return n + fill;
}
template <bool FILL, typename T, int BATCH, bool PER_CHUNK>
__device__ __forceinline__ void make_streams(const RoundLds<BATCH, PER_CHUNK>& s, T (*stream)[BATCH], int unit,
                                             bool split, bool by_chunk, int wv, int lane, int (&n)[kGroups]) {
  constexpr int kChunks = RoundLds<BATCH, PER_CHUNK>::chunks;
  static_assert(kChunks <= kGroups, "n holds one end per chunk");
  const uint64_t mine = (&s.mask[wv][0][0])[lane < kGroups * kChunks ? lane : 0];
  auto put = [&](int g, int c, int at) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)mine, g * kChunks + c);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(mine >> 32), g * kChunks + c);
    const uint64_t m = (uint64_t)lo | ((uint64_t)hi << 32);
    if (__builtin_amdgcn_inverse_ballot_w64(m))
      stream[g][at + (int)__builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, 0u))] =
          (T)((c * kWave + lane) * unit);
    return (int)__popcll(m);
  };
  if constexpr (!FILL) {
    if (lane < kGroups) stream[lane][0] = 0;
    wave_sync();
  }
  if (by_chunk) {
    int at = 0;
#pragma unroll
    for (int c = 0; c < kGroups; ++c) {
      if (c < kChunks) {
        at += put(0, c, at);
        if constexpr (FILL) at = fill_four(stream[0], at, lane);
      }
      n[c] = at;
    }
  } else {
#pragma unroll
    for (int g = 0; g < kGroups; ++g) {
      n[g] = 0;
      if (split && g > 0) continue;
#pragma unroll
      for (int c = 0; c < kChunks; ++c) n[g] += put(g, c, n[g]);
    }
  }
  wave_sync();
}
template <typename T>
__device__ __forceinline__ T lds_at(const T* base, uint32_t bytes) {
  return *reinterpret_cast<const T*>(reinterpret_cast<const char*>(base) + bytes);
}

// Row-parallel forward: of the entries in [from, until) of the stream, one
// chunk's, those that meet the rectangle of the pixels `bits` of the group at
// (gx, gy) move to its front, the rest becomes kNoEntry.
__device__ __forceinline__ void retest_chunk(uint16_t* stream, int from, int until, const float4* s_r0,
                                             const float4* s_r1, const float4* s_r2, const int32_t* __restrict__ bin,
                                             uint32_t bits, int32_t ix0, int32_t iy0, int32_t gx, int32_t gy, int lane,
                                             float log2_alpha_min) {
  const bool slot = from + lane < until;
  const uint32_t off = slot ? stream[from + lane] : kNoEntry;
  bool rel = off != kNoEntry;
  if (rel) {
    const Rect rg = group_rect(bits, gx, gy);
    const uint32_t r = __float_as_uint(lds_at(s_r2, off).w);  // a stream holds valid entries only
    const int2 box = *reinterpret_cast<const int2*>(bin + 4 * (int64_t)r);
    const EntryTest t = entry_test(lds_at(s_r0, off), lds_at(s_r1, off), ix0, iy0, log2_alpha_min);
    rel = box_meets(box, ix0 + rg.x0, ix0 + rg.x1, iy0 + rg.y0, iy0 + rg.y1) &&
          group_meets(t, (float)rg.x0, (float)rg.x1, (float)rg.y0, (float)rg.y1);
  }
  const uint64_t m = __builtin_amdgcn_ballot_w64(rel);
  // each lane of a slot writes one: the entries in order, then the empty ones
  const int below = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
  wave_sync();
  if (slot) stream[from + (rel ? below : (int)__popcll(m) + lane - below)] = (uint16_t)(rel ? off : kNoEntry);
  wave_sync();
}
__device__ __forceinline__ int max4(const int (&n)[kGroups]) {
  const int a = n[0] > n[1] ? n[0] : n[1], b = n[2] > n[3] ? n[2] : n[3];
  return a > b ? a : b;
}

// Work item of a render workgroup.  With a tile order (longest lists first),
// each of the first kSplitTiles tiles of the order gets four workgroups.  If
// the tile splits, they take one 8x8 quarter each, with one 4x4 pixel group
// per wave, so the tile's sixteen groups walk their streams independently
// instead of four to a wave in lockstep: the longest lists set the kernels'
// length.  Otherwise one of the four takes the whole tile and the other three
// exit.  The four blocks of a tile are b, b + 8, b + 16, b + 24 of a run of
// 32: they run on one XCD (block b runs on XCD b mod 8) and share its L2, so
// the tile's records are fetched from HBM once.  The whole-tile runner is the
// tile's block with quarter index (b >> 5) & 3, rotating from run to run: an
// XCD places its workgroups on its CUs in turn, and a fixed runner would put
// every runner on every fourth CU while the others got only the exiting
// blocks (measured: forward-only renders 1.7x slower).
//
// Backward: a tile splits when its list has at least kSplitLen entries; a
// split wave's four rows hold the same 16 pixels and take four consecutive
// entries of the group's stream per step, combined across rows by scans.
// Forward: the row-parallel form costs about twice the instructions per
// (entry, group) of a whole-tile wave, so it only pays when the work is
// concentrated in few tiles.  When at least half of the tiles are empty (the
// tile at the middle of the order has no entries) every tile of at least
// kSplitLen entries splits row-parallel; otherwise only the kFwdSpreadTiles
// longest split, when they reach kFwdSpreadLen entries, with the group in
// lanes 0-15.
constexpr int32_t kSplitTiles = 2048;
constexpr uint32_t kSplitLen = 128;
constexpr int32_t kFwdSpreadTiles = 256;
constexpr uint32_t kFwdSpreadLen = 2048;
struct WorkItem {
  int32_t tile;
  int32_t quarter;  // -1: whole tile
  bool skip;
  bool rowpar;      // split with the rows as consecutive entries
};
__device__ __forceinline__ WorkItem work_item(const uint32_t* order, const uint32_t* ranges, int32_t nsplit,
                                              int32_t tiles_total, bool forward) {
  WorkItem w{(int32_t)blockIdx.x, -1, false, false};
  if (order == nullptr) return w;
  const int32_t b = (int32_t)blockIdx.x;
  if (b < 4 * nsplit) {
    const int32_t t = ((b >> 5) << 3) + (b & 7);
    w.tile = (int32_t)uload(order + t);
    const uint32_t len = uload(ranges + 2 * w.tile + 1) - uload(ranges + 2 * w.tile);
    const int32_t q = (b >> 3) & 3;
    bool split = len >= kSplitLen, rowpar = true;
    if (forward) {
      const uint32_t mid = uload(order + tiles_total / 2);
      const bool concentrated = uload(ranges + 2 * mid + 1) == uload(ranges + 2 * mid);
      if (!concentrated) {
        split = t < kFwdSpreadTiles && len >= kFwdSpreadLen;
        rowpar = false;
      }
    }
    if (split) {
      w.quarter = q;
      w.rowpar = rowpar;
    } else {
      w.skip = q != ((b >> 5) & 3);
    }
  } else {
    // Workgroups go to the eight XCDs in turn.  Inside each aligned group of
    // 64 workgroups, the eight of one XCD take eight consecutive entries of
    // the order (neighbouring tiles of one length class, which share records,
    // in one L2); every XCD still walks the order at the same pace.  Partial
    // groups at either end keep the identity, so the map stays a bijection.
    int32_t p = b;
    const int32_t g0 = b & ~63, lo = 4 * nsplit, hi = (int32_t)gridDim.x;
    if (g0 >= lo && g0 + 64 <= hi) p = g0 + ((b & 7) << 3) + ((b & 63) >> 3);
    w.tile = (int32_t)uload(order + (p - 3 * nsplit));
  }
  return w;
}
// Pixel of this lane and the origin of its 4x4 group (see work_item).  In a
// split work item the four rows of a wave carry the same 16 pixels.
struct LanePixel {
  int32_t sx0, sy0;  // origin of group 0 of this wave
  int32_t px, py;
  bool on;           // lane carries a pixel of the work item
};
__device__ __forceinline__ LanePixel lane_pixel(int32_t tx, int32_t ty, int32_t quarter, int wv, int lane,
                                                bool rows_share) {
  LanePixel l;
  if (quarter < 0) {
    const int grp = lane >> 4;
    l.sx0 = tx * kTile + (wv & 1) * 8;
    l.sy0 = ty * kTile + (wv >> 1) * 8;
    l.px = l.sx0 + (grp & 1) * 4 + (lane & 3);
    l.py = l.sy0 + (grp >> 1) * 4 + ((lane >> 2) & 3);
    l.on = true;
  } else {
    l.sx0 = tx * kTile + (quarter & 1) * 8 + (wv & 1) * 4;
    l.sy0 = ty * kTile + (quarter >> 1) * 8 + (wv >> 1) * 4;
    l.px = l.sx0 + (lane & 3);
    l.py = l.sy0 + ((lane >> 2) & 3);
    l.on = rows_share || lane < 16;  // rows = consecutive entries of the group's stream, or lanes 0-15 only
  }
  return l;
}
// Tiles of the order that get four workgroups: a multiple of 8 (see work_item).
inline int32_t split_tiles(const uint32_t* order, int32_t tiles_total) {
  const int32_t t = tiles_total < kSplitTiles ? tiles_total : kSplitTiles;
  return order ? t & ~7 : 0;
}

constexpr int kFwdUnroll = 2;   // entries of a group's stream per forward iteration
static_assert(kFwdUnroll == 2, "an iteration's two 16-bit offsets come from one 32-bit read");
constexpr uint32_t kNoOffset = 0xffffffffu, kNoRecord = 0xffffffffu;

// Work per tile spans four orders of magnitude and a wave's list is walked in
// order, so the longest lists set the kernel's length.  Waves of long lists
// get a higher issue priority than the waves sharing their SIMD.
__device__ __forceinline__ void set_wave_priority(uint32_t list_len) {
  if (list_len >= 2048) __builtin_amdgcn_s_setprio(3);
  else if (list_len >= 1024) __builtin_amdgcn_s_setprio(2);
  else if (list_len >= 512) __builtin_amdgcn_s_setprio(1);
}

// Forward.  Per round the workgroup gathers up to 256 consecutive list entries
// (index, pixel box, 48-byte record) into LDS with one load per thread, so the
// latency of the random record gathers is paid once per 256 entries; all
// threads test them against the workgroup's pixel groups (test_round), and
// each wave walks the lists of its own groups with broadcast LDS loads.
// Bound by the vector instructions of the walk, and under row-parallel
// splitting by the latency of the longest lists.  Measured with the tests in
// the staging thread, one list per round, the weights summed before they go to
// LDS and 72 registers instead of 79 (seven waves per SIMD without
// accumulation): 3M Gaussians at 1920x1080 with accumulation 599 -> 549 us and
// without 340 -> 333 us, 100k at 637x479 with accumulation 126 -> 64 us, 4 views
// of 1.5M 745 -> 707 us.  With the walk's decisions as wave masks (62 vector
// instructions per two entries instead of 78) the last 64 -> 61 and 712 -> 642 us,
// 3M without accumulation 333 -> 305 us, 16 views of 1M 2517 -> 2279 us.
template <bool ACC, bool OUT, int DEPTH>
__global__ __launch_bounds__(kBlock) void k_render_fwd(const float* __restrict__ rec, const int32_t* __restrict__ bin,
                                                       const uint32_t* __restrict__ vals,
                                                       const uint32_t* __restrict__ ranges,
                                                       const uint32_t* __restrict__ order, int32_t nsplit, int64_t n,
                                                       const float* __restrict__ means,
                                                       const float* __restrict__ scales,
                                                       const float* __restrict__ quats, FwdOut o, KOpts op,
                                                       int32_t per_view, ViewSet vs) {
  // s_r2[k].w carries the record index (the forward never reads the opacity
  // field), so one read returns colour and index
  __shared__ float4 s_r0[kFwdBatch], s_r1[kFwdBatch], s_r2[kFwdBatch];
  __shared__ RoundLds<kFwdBatch, false> s_round;
  __shared__ float s_z[DEPTH == GS_DEPTH_BLEND ? kFwdBatch : 1];
  // per staged entry: importance and max weight gathered from the whole
  // workgroup with LDS atomics, flushed with one global atomic per entry
  // (double, and one lane per group: see row_sum_max2)
  __shared__ double s_acc_w[ACC ? kFwdBatch : 1];
  __shared__ uint32_t s_acc_m[ACC ? kFwdBatch : 1];
  __shared__ alignas(4) uint16_t s_stream[kWaves][kGroups][kFwdBatch];
  // an offset read past a stream's end is unused, but it is read: keep it in range
  for (int q = threadIdx.x; q < kWaves * kGroups * kFwdBatch / 2; q += kBlock)
    reinterpret_cast<AliasedU32*>(&s_stream[0][0][0])[q] = 0;
  const WorkItem wi = work_item(order, ranges, nsplit, vs.tiles_total, true);
  if (wi.skip) return;
  const int32_t tile = wi.tile;
  const int32_t v = view_of_tile(vs, tile);
  const KView& cam = vs.v[v];
  const int32_t lt = tile - cam.tile_base;
  const int32_t tx = lt % cam.tiles_x, ty = lt / cam.tiles_x;
  // Lanes: a wave owns an 8x8 quarter of the tile as four 4x4 pixel groups,
  // one group per 16-lane row (lane = 16 g + 4 y + x), or, for a split heavy
  // tile, one 4x4 group in lanes 0-15.  Each group walks its own stream of
  // entries (those meeting its still-compositing pixels), so a wave iterates
  // max over groups instead of the union of the four streams.
  const int wv = (int)uniform_u32(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int grp = lane >> 4;
  const bool rp = wi.quarter >= 0 && wi.rowpar;  // split work item: rows are consecutive entries
  const LanePixel lp = lane_pixel(tx, ty, wi.quarter, wv, lane, rp);
  const int32_t sx0 = lp.sx0, sy0 = lp.sy0;
  const bool inside = lp.on && lp.px < cam.width && lp.py < cam.height;
  const float pxc = (float)lp.px + 0.5f, pyc = (float)lp.py + 0.5f;
  const uint32_t start = uload(ranges + 2 * tile), end = uload(ranges + 2 * tile + 1);
  const int64_t vbase = (int64_t)v * n;
  const int64_t nrec = (int64_t)vs.count * n;
  set_wave_priority(end - start);
  float T = 1.f, c0 = 0.f, c1 = 0.f, c2 = 0.f, wbest = 0.f, dblend = 0.f;
  uint32_t best = kNoRecord;  // record index
  uint32_t lastpos = 0, cnt = 0;
  // split work items: list position of `best`; others: LDS offset of the last
  // entry of this round that the pixel has composited
  uint32_t at = kNoOffset;
  bool done = !inside;
  // Staging pipeline: while round R is processed, the records of round R + 1
  // and the list indices of round R + 2 are already in flight.
  Staged cur = fetch_entry(rec, bin, start + threadIdx.x < end ? vals[start + threadIdx.x] : 0u,
                           start + threadIdx.x < end, nrec);
  uint32_t nidx = start + kFwdBatch + threadIdx.x < end ? vals[start + kFwdBatch + threadIdx.x] : 0u;
  const int32_t ix0 = tx * kTile + (wi.quarter > 0 ? (wi.quarter & 1) * 8 : 0);
  const int32_t iy0 = ty * kTile + (wi.quarter > 0 ? (wi.quarter >> 1) * 8 : 0);
  const bool split = wi.quarter >= 0;
  for (uint32_t base = start; base < end; base += kFwdBatch) {
    const uint32_t tid = (uint32_t)fresh((int)threadIdx.x);
    const uint64_t am = __builtin_amdgcn_ballot_w64(!done);
    if (lane == 0) s_round.active[wv][0] = am;
    __syncthreads();  // also orders this round's LDS writes after the last round's reads
    if (s_round.none_active()) break;
    const uint32_t count = (end - base) < (uint32_t)kFwdBatch ? (end - base) : (uint32_t)kFwdBatch;
    s_r0[tid] = cur.r0;
    s_r1[tid] = cur.r1;
    const bool entry = cur.entry();
    s_r2[tid] = make_float4(entry ? cur.r2.x : 0.f, entry ? cur.r2.y : 0.f, entry ? cur.r2.z : 0.f,
                            __uint_as_float(cur.idx));
    if (DEPTH == GS_DEPTH_BLEND) s_z[tid] = entry ? cur.z : 0.f;
    if (ACC) {
      const int zero = fresh(0);
      s_acc_w[tid] = __hiloint2double(zero, zero);
      s_acc_m[tid] = 0u;
    }
    test_round(s_round, nullptr, 0u, split, fresh_uniform(ix0), fresh_uniform(iy0), cur.box, cur.r0, cur.r1, (uint32_t)tid < count, wv,
               fresh(lane), op.log2_alpha_min);
    __syncthreads();
    {
      const uint32_t jn = base + kFwdBatch + tid, jnn = jn + kFwdBatch;
      cur = fetch_entry(rec, bin, nidx, jn < end, nrec);
      nidx = jnn < end ? vals[jnn] : 0u;
    }
    if (!rp) at = kNoOffset;
    if (am != 0) {  // some pixel of this wave still composites
      int n4[kGroups];
      make_streams<true>(s_round, s_stream[wv], 16, split, rp, wv, fresh(lane), n4);
      // Split work item: row r takes the r-th of the next four entries of the
      // group's stream.  The transmittance in front of each is T times the
      // product of (1 - alpha) over the rows before it; an entry is composited
      // unless its own or an earlier row's entry reaches the stop.  Each row
      // keeps partial colour, depth, count and argmax, merged at the end.
      // Each four is of one chunk of 64 staged entries, and a chunk's entries
      // are those that meet the pixels compositing at its start: which entries
      // share a product (and with it the rounding of the transmittance) does
      // not depend on how many entries a round has.  Two fours per iteration:
      // their records are read and their alphas and products formed side by
      // side, then they are composited in order.
      // What decides (which lanes pass, stop, are done) is kept as wave masks in
      // scalar registers: only the comparisons are vector instructions.
      uint64_t stopped = __builtin_amdgcn_ballot_w64(done);
      uint64_t met = am;  // pixels that the rest of the stream was tested against
#pragma unroll 1
      for (int i = 0; rp && i < n4[3];) {
        const int row = (fresh((int)threadIdx.x) & 63) >> 4;
        const uint64_t now = ~stopped;
        if (now == 0) break;
        if (now != met) {  // rare: some pixel has stopped in the chunk that ended here
          for (int from = i; from < n4[3];) {
            const int end = from < n4[1] ? n4[1] : from < n4[2] ? n4[2] : n4[3];
            retest_chunk(s_stream[wv][0], from, end, s_r0, s_r1, s_r2, bin, (uint32_t)now & 0xffffu,
                         fresh_uniform(ix0), fresh_uniform(iy0), (wv & 1) * 4, (wv >> 1) * 4, fresh(lane),
                         op.log2_alpha_min);
            from = end;
          }
          met = now;
        }
        int until = n4[3];
        const uint16_t* sp = &s_stream[wv][0][i + row];
#pragma unroll 1
        for (; i < until; i += 2 * kGroups, sp += 2 * kGroups) {
          uint32_t off[2];
          uint64_t pass[2];
          float4 q2[2];
          float al[2], om[2], wg[2];
          RowScan tf[2];
#pragma unroll
          for (int u = 0; u < 2; ++u) {
            const uint32_t entry = i + u * kGroups < until ? (uint32_t)sp[u * kGroups] : kNoEntry;
            const bool hr = entry != kNoEntry;
            off[u] = hr ? entry : 0u;
            const float4 r0 = lds_at(s_r0, off[u]), r1 = lds_at(s_r1, off[u]);
            q2[u] = lds_at(s_r2, off[u]);
            const float dx = (pxc - r0.x) - r0.z, dy = (pyc - r0.y) - r0.w;
            const float ee = r1.w - (r1.x * dx * dx + r1.y * dx * dy + r1.z * dy * dy);
            al[u] = fminf(op.alpha_max, __builtin_amdgcn_exp2f(ee));
            pass[u] = __builtin_amdgcn_ballot_w64(entry != kNoEntry) & ~stopped &
                      __builtin_amdgcn_ballot_w64(ee >= op.log2_alpha_min);
            om[u] = __builtin_amdgcn_inverse_ballot_w64(pass[u]) ? 1.f - al[u] : 1.f;
            tf[u] = rows_scan_mul(om[u], row);
          }
#pragma unroll
          for (int u = 0; u < 2; ++u) asm("" : "+v"(q2[u].w));
#pragma unroll
          for (int u = 0; u < 2; ++u) {
            const uint64_t sb = pass[u] & __builtin_amdgcn_ballot_w64(T * tf[u].incl < op.t_min);
            uint64_t in = pass[u];
            float Tn = T * tf[u].total;
            if (sb != 0ull) {
              // rare: some pixel stops at one of these entries; later rows of its
              // column are dropped and its transmittance is the one in front of
              // the stopping entry
              const int l = fresh(lane);
              const uint64_t col = 0x0001000100010001ull << (l & 15);
              const bool earlier = (sb & col & ((1ull << (l & 48)) - 1ull)) != 0;
              in = pass[u] & ~sb & ~__builtin_amdgcn_ballot_w64(earlier);
              Tn = T * rows_scan_mul(__builtin_amdgcn_inverse_ballot_w64(in) ? om[u] : 1.f, row).total;
              const uint64_t columns = (sb | (sb >> 16) | (sb >> 32) | (sb >> 48)) & 0xffffull;
              stopped |= columns * 0x0001000100010001ull;
              // the walk leaves off at the end of this chunk, which may be
              // between the two fours (row 0 of a four always has an entry)
              const uint32_t chunk = uniform_u32(off[u]) / (16u * kWave);
              until = chunk == 0 ? n4[0] : chunk == 1 ? n4[1] : chunk == 2 ? n4[2] : n4[3];
              if (u == 0) {
                pass[1] = i + kGroups < until ? pass[1] & ~stopped : 0ull;
                om[1] = __builtin_amdgcn_inverse_ballot_w64(pass[1]) ? om[1] : 1.f;
                tf[1] = rows_scan_mul(om[1], row);
              }
            }
            const bool inc = __builtin_amdgcn_inverse_ballot_w64(in);
            const float wgt = inc ? al[u] * (T * tf[u].excl) : 0.f;
            c0 += wgt * q2[u].x;
            c1 += wgt * q2[u].y;
            c2 += wgt * q2[u].z;
            if (DEPTH == GS_DEPTH_BLEND) dblend += wgt * lds_at(s_z, off[u] >> 2);
            const uint32_t pos = base + (off[u] >> 4) - start;
            const bool better = wgt > wbest;  // a row's entries arrive in order: the nearer wins ties
            wbest = better ? wgt : wbest;
            best = better ? __float_as_uint(q2[u].w) : best;
            at = better ? pos : at;
            lastpos = inc ? pos + 1 : lastpos;
            cnt += inc ? 1u : 0u;
            wg[u] = wgt;
            T = Tn;
          }
          if (ACC) {
            const SumMax r = row_sum_max2(wg[0], wg[1]);
            if ((lane & 7) == 0 && r.max > 0.f) {
              const uint32_t k = ((lane & 8) ? off[1] : off[0]) >> 4;
              atomicAdd(&s_acc_w[k], (double)r.sum);
              atomicMax(&s_acc_m[k], __float_as_uint(r.max));
            }
          }
        }
        i = until;
      }
      // kFwdUnroll entries of the group's stream per iteration: their records
      // are read and their alphas evaluated side by side, then they are
      // composited in order (each sees the previous one's transmittance and
      // stop), so the result is that of one-by-one compositing with a fraction
      // of the loop latency.  The offsets of the next iteration are read ahead.
      const int group = (fresh((int)threadIdx.x) & 63) >> 4;
      int mine = group == 0 ? n4[0] : group == 1 ? n4[1] : group == 2 ? n4[2] : n4[3];
      const int longest = (int)uniform_u32((uint32_t)(rp ? 0 : max4(n4)));
      const uint16_t* stream = &s_stream[wv][group][0];
      uint32_t pair = *reinterpret_cast<const AliasedU32*>(stream);
      for (int i = 0; i < longest; i += kFwdUnroll) {
        uint32_t off[kFwdUnroll];
        uint64_t has[kFwdUnroll];
#pragma unroll
        for (int u = 0; u < kFwdUnroll; ++u) {
          has[u] = __builtin_amdgcn_ballot_w64(i + u < mine);
          off[u] = (pair >> (16 * u)) & 0xffffu;
        }
        const int next = i + kFwdUnroll < kFwdBatch ? i + kFwdUnroll : i;
        pair = *reinterpret_cast<const AliasedU32*>(stream + next);
        float4 q2[kFwdUnroll];
        float al[kFwdUnroll], ee[kFwdUnroll], wg[kFwdUnroll];
#pragma unroll
        for (int u = 0; u < kFwdUnroll; ++u) {
          const float4 r0 = lds_at(s_r0, off[u]), r1 = lds_at(s_r1, off[u]);
          q2[u] = lds_at(s_r2, off[u]);
          const float dx = (pxc - r0.x) - r0.z, dy = (pyc - r0.y) - r0.w;
          ee[u] = r1.w - (r1.x * dx * dx + r1.y * dx * dy + r1.z * dy * dy);
          al[u] = fminf(op.alpha_max, __builtin_amdgcn_exp2f(ee[u]));
        }
        // (the index is read with the colour, not again where the weight is the largest)
#pragma unroll
        for (int u = 0; u < kFwdUnroll; ++u) asm("" : "+v"(q2[u].w));
        uint64_t stops = 0;
#pragma unroll
        for (int u = 0; u < kFwdUnroll; ++u) {
          // Branch-free per lane: selects keep the state of lanes that skip the
          // entry or have stopped (staged colours are finite, so adding a zero
          // weight leaves the colour unchanged).
          const uint64_t pass = has[u] & ~stopped & __builtin_amdgcn_ballot_w64(ee[u] >= op.log2_alpha_min);
          const float Tn = T * (1.f - al[u]);
          const uint64_t stop = pass & __builtin_amdgcn_ballot_w64(Tn < op.t_min);
          const bool inc = __builtin_amdgcn_inverse_ballot_w64(pass & ~stop);
          stopped |= stop;
          stops |= stop;
          const float wgt = inc ? al[u] * T : 0.f;
          T = inc ? Tn : T;
          c0 += wgt * q2[u].x;
          c1 += wgt * q2[u].y;
          c2 += wgt * q2[u].z;
          if (DEPTH == GS_DEPTH_BLEND) dblend += wgt * lds_at(s_z, off[u] >> 2);
          const bool better = wgt > wbest;  // strict: the nearer entry wins ties
          wbest = better ? wgt : wbest;
          best = better ? __float_as_uint(q2[u].w) : best;
          at = inc ? off[u] : at;
          cnt += inc ? 1u : 0u;
          wg[u] = wgt;
        }
        if (ACC) {
          const SumMax r = row_sum_max2(wg[0], wg[1]);
          if ((lane & 7) == 0 && r.max > 0.f) {
            const uint32_t k = ((lane & 8) ? off[1] : off[0]) >> 4;
            atomicAdd(&s_acc_w[k], (double)r.sum);
            atomicMax(&s_acc_m[k], __float_as_uint(r.max));  // weights are >= 0: bit patterns have their order
          }
        }
        if (stops != 0) {
          // a group whose pixels have all stopped drops the rest of its stream
          if (stopped == ~0ull) break;
          if (((stopped >> (16 * group)) & 0xffffull) == 0xffffull) mine = 0;
        }
      }
      done = __builtin_amdgcn_inverse_ballot_w64(stopped);
    }
    if (!rp && at != kNoOffset) lastpos = base - start + (at >> 4) + 1;
    if (ACC) {
      __syncthreads();
      const uint32_t ft = (uint32_t)fresh((int)threadIdx.x);
      if (ft < count && s_acc_m[ft] != 0u) {
        const uint32_t r = __float_as_uint(s_r2[ft].w);
        const int64_t ai = per_view ? (int64_t)r : (int64_t)r - vbase;
        if (o.imp) atomicAdd(o.imp + ai, (float)s_acc_w[ft]);
        if (o.wmax) atomicMax(reinterpret_cast<unsigned int*>(o.wmax) + ai, s_acc_m[ft]);
      }
    }
  }
  if (rp) {
    // merge the rows' partials (every row of a column holds the same pixel)
    c0 = rows_sum(c0);
    c1 = rows_sum(c1);
    c2 = rows_sum(c2);
    if (DEPTH == GS_DEPTH_BLEND) dblend = rows_sum(dblend);
    cnt = rows_sum_u32(cnt);
    lastpos = rows_max_u32(lastpos);
    // argmax: the larger weight, on equal weights the earlier list position
#pragma unroll
    for (int step = 0; step < 2; ++step) {
      const RowsTwo w = step == 0 ? rows_pair(__float_as_uint(wbest)) : rows_halves(__float_as_uint(wbest));
      const RowsTwo b = step == 0 ? rows_pair(best) : rows_halves(best);
      const RowsTwo q = step == 0 ? rows_pair(at) : rows_halves(at);
      const float wa = __uint_as_float(w.a), wb = __uint_as_float(w.b);
      const bool take_b = wb > wa || (wb == wa && q.b < q.a);
      wbest = take_b ? wb : wa;
      best = take_b ? b.b : b.a;
      at = take_b ? q.b : q.a;
    }
    if (lane >= 16) return;  // row 0 writes the pixel
  }
  const LanePixel le = lane_pixel(tx, ty, wi.quarter, wv, fresh(lane), rp);
  const int32_t px = le.px, py = le.py;
  if (!le.on || px >= cam.width || py >= cam.height) return;
  const int32_t gbest = best == kNoRecord ? -1 : (int32_t)((int64_t)best - vbase);
  if (ACC && o.area && gbest >= 0) atomicAdd(o.area + (per_view ? vbase + gbest : (int64_t)gbest), 1u);
  if (!OUT) return;
  const int64_t P = vs.pixels_total;
  const int64_t gp = cam.pixel_base + (int64_t)py * cam.width + px;
  o.color[gp] = c0 + T * op.bg[0];
  o.color[P + gp] = c1 + T * op.bg[1];
  o.color[2 * P + gp] = c2 + T * op.bg[2];
  o.t_final[gp] = T;
  o.last[gp] = lastpos;
  o.imax[gp] = gbest;
  if (o.n_contrib) o.n_contrib[gp] = cnt;
  float dep = 0.f;
  uint8_t h = 0;
  if (gbest >= 0 && (o.depth || o.hit)) {
    RayCam rc;
    for (int k = 0; k < 9; ++k) rc.R[k] = cam.R[k];
    for (int k = 0; k < 3; ++k) rc.t[k] = cam.t[k];
    rc.fx = cam.fx; rc.fy = cam.fy; rc.cx = cam.cx; rc.cy = cam.cy;
    const MidDepth md = mid_depth(rc, means, scales, quats, n, gbest, pxc, pyc);
    const float dm = md.depth;
    h = (uint8_t)md.hit;
    if (DEPTH == GS_DEPTH_MID) dep = dm;
    else if (DEPTH == GS_DEPTH_CENTER) dep = rec[(vbase + gbest) * kRecFloats + 12];
    else dep = dblend;
  }
  if (o.depth) o.depth[gp] = dep;
  if (o.hit) o.hit[gp] = h;
}

// ---------------------------------------------------------------------------
// backward
// ---------------------------------------------------------------------------
// One list entry for the backward: the first 48 bytes of its record, with the
// opacity negated for an inactive entry (a drawn record's opacity is positive),
// so the walk needs no separate flag.  Where there is no entry or its index is
// corrupt (outside this view's records): an inactive one of zeros with an empty
// box, so that past a stream's end, too, every product with a weight of 0 is 0.
struct StagedB {
  int2 box;
  float4 r0, r1, r2;
};
template <bool MASKED>
__device__ __forceinline__ StagedB fetch_entry_bwd(const float* __restrict__ rec, const int32_t* __restrict__ bin,
                                                   const uint8_t* __restrict__ active, uint32_t r, bool in_list,
                                                   int64_t nrec, int64_t vbase) {
  StagedB e;
  const bool valid = in_list && (int64_t)r < nrec && (int64_t)r >= vbase;
  r = valid ? r : (uint32_t)vbase;
  const bool act = valid && (!MASKED || active[(int64_t)r - vbase] != 0);
  e.box = valid ? *reinterpret_cast<const int2*>(bin + 4 * (int64_t)r) : make_int2(0xffff, 0xffff);
  e.r0 = e.r1 = e.r2 = make_float4(0.f, 0.f, 0.f, 0.f);
  if (valid) {
    const float4* R4 = reinterpret_cast<const float4*>(rec + (int64_t)r * kRecFloats);
    e.r0 = R4[0];
    e.r1 = R4[1];
    e.r2 = R4[2];
  }
  e.r2.w = act ? fabsf(e.r2.w) : -fabsf(e.r2.w);
  return e;
}

// The nine sums of an entry over each 16-lane row (4x4 pixels): of six per-lane
// partials p, and of the weight w times the three channels of dL/dcolour.
//
// Partials: lanes 1 apart, 2 apart, 8 apart, 4 apart.  The first two steps keep
// one of two values in either lane (selects), the third one of two registers in
// either half of the row, chosen by the bank mask of the add itself (lanes of a
// disabled bank keep the register's value), which the compiler cannot express:
// hence the assembly.  The last, a rotate by 4, is right where bit 2 of the lane
// is set.  Halves first, all by bank masks, takes 13 instructions instead of 16
// and was not kept: the gradient of a needle's scales is a difference of the
// second moments smaller than they are by the square of its elongation, so it
// shows every rounding in which the three differ, and another tree (with the
// scalar suffix, see alpha_gradient) moved it by three times the noise of the
// atomics.  Channels: lane m of a quad sums channel m over the quad's pixels, w
// of each pixel by a broadcast inside the quad times that pixel's channel m (gm,
// the same for all entries), then the four quads are added: six instructions
// instead of three products and ten.  A DPP read needs two instructions after
// the write of its register; the order below keeps that distance.  Returned: in
// lane L of a row the total of value sum_slot(L), where that is not negative.
__device__ __forceinline__ int sum_slot(int lane) {
  const int l = lane & 15;
  if (l & 4) return l < 8 ? l - 4 : l < 14 ? l - 8 : -1;
  return l < 3 ? 6 + l : -1;
}
struct ChannelPixels {
  float x[4];  // lane m of a quad: channel m of the quad's pixels
};
__device__ __forceinline__ ChannelPixels channel_pixels(float g0, float g1, float g2, int lane) {
  ChannelPixels r;
  const int m = lane & 3;
#define MS_QUAD(k, ctrl) \
  { \
    const float a = dpp_take<ctrl>(g0), b = dpp_take<ctrl>(g1), c = dpp_take<ctrl>(g2); \
    r.x[k] = m == 0 ? a : m == 1 ? b : m == 2 ? c : 0.f; \
  }
  MS_QUAD(0, 0x00)
  MS_QUAD(1, 0x55)
  MS_QUAD(2, 0xAA)
  MS_QUAD(3, 0xFF)
#undef MS_QUAD
  return r;
}
__device__ __forceinline__ float row_sum9(const float (&p)[6], float w, const ChannelPixels& gm, int lane) {
  constexpr int kXor1 = 0xB1, kXor2 = 0x4E;
  const bool odd = (lane & 1) != 0, upper = (lane & 2) != 0;
  float a[3];
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    const float keep = odd ? p[2 * j + 1] : p[2 * j], send = odd ? p[2 * j] : p[2 * j + 1];
    a[j] = keep + dpp_take<kXor1>(send);
  }
  const float b = (upper ? a[1] : a[0]) + dpp_take<kXor2>(upper ? a[0] : a[1]);
  const float c = a[2] + dpp_take<kXor2>(a[2]);
  float d, h;
  asm("s_nop 1\n\t"
      "v_mul_f32_dpp %1, %4, %5 quad_perm:[0,0,0,0] row_mask:0xf bank_mask:0xf\n\t"
      "v_add_f32_dpp %0, %2, %2 row_ror:8 row_mask:0xf bank_mask:0x3\n\t"
      "v_fmac_f32_dpp %1, %4, %6 quad_perm:[1,1,1,1] row_mask:0xf bank_mask:0xf\n\t"
      "v_add_f32_dpp %0, %3, %3 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
      "v_fmac_f32_dpp %1, %4, %7 quad_perm:[2,2,2,2] row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f32_dpp %1, %4, %8 quad_perm:[3,3,3,3] row_mask:0xf bank_mask:0xf\n\t"
      "v_add_f32_dpp %0, %0, %0 row_ror:4 row_mask:0xf bank_mask:0xf\n\t"
      "s_nop 0\n\t"
      "v_add_f32_dpp %1, %1, %1 row_ror:8 row_mask:0xf bank_mask:0xf\n\t"
      "s_nop 1\n\t"
      "v_add_f32_dpp %1, %1, %1 row_ror:4 row_mask:0xf bank_mask:0xf"
      : "=&v"(d), "=&v"(h)
      : "v"(b), "v"(c), "v"(w), "v"(gm.x[0]), "v"(gm.x[1]), "v"(gm.x[2]), "v"(gm.x[3]));
  return (lane & 4) != 0 ? d : h;
}

// dL/dalpha of one entry of a pixel, with the transmittance T in front of it,
// 1 / (1 - alpha) and the colour composited behind it, channel by channel.  The
// suffix as one scalar (its product with dL/dcolour) saves six instructions and,
// in split work items, two of the three scans; not kept for the reason row_sum9
// gives (it also turns an infinite dL/dcolour times a zero background into NaN).
__device__ __forceinline__ float alpha_gradient(const float (&g)[3], float4 c, float T, float iom, const float (&s)[3]) {
  const float x0 = __builtin_fmaf(c.x, T, -(s[0] * iom));
  const float x1 = __builtin_fmaf(c.y, T, -(s[1] * iom));
  const float x2 = __builtin_fmaf(c.z, T, -(s[2] * iom));
  return __builtin_fmaf(g[2], x2, __builtin_fmaf(g[0], x0, g[1] * x1));
}

// The nine sums of an entry over pixels, with e = dL/dalpha alpha (0 where
// alpha is clamped or the entry is not composited) and w the weight:
//   0, 1: sum e (2 A dx + B dy), e (B dx + 2 C dy)
//   2, 3, 4: sum e dx dx, e dx dy, e dy dy
//   5: sum e               6, 7, 8: sum w dL/dcolour
// with the staged conic (A, B, C), log2(e) / 2 times the conic with B twice its
// off-diagonal.  What else the 2D gradient adds to them is constant per record,
// so it is applied once to the sums: the record's gradient is (ln 2 S0, ln 2 S1,
// -S2 / 2, -S3, -S4 / 2, S5 / opacity, S6, S7, S8).  The conic stays inside the
// first two: for a needle 2 A dx + B dy cancels by its elongation, and taken of
// the sums instead of per pixel it magnified their rounding (error of the means
// against 64 bits 4 to 7 % larger at elongations of 10 to 32; five vector
// instructions per walked entry).
__device__ __forceinline__ float g2d_component(int c, float x, float opacity) {
  constexpr float kLn2 = 0.6931471805599453f;
  const float scale = c < 2 ? kLn2 : c == 5 ? __builtin_amdgcn_rcpf(opacity) : c > 5 ? 1.f : c == 3 ? -1.f : -0.5f;
  return scale * x;
}

// One group's sums of one entry leave the row from nine of its lanes: into the
// entry's accumulators in LDS, which the workgroup adds to the record's 2D
// gradient once per round, or (deterministic reduction) into the entry's slot
// for this group (list position j, group g16 of the tile's sixteen 4x4
// groups), marked in the entry's mask.  A slot is written at most once: each
// group walks an entry at most once.  LDS adds floats one lane at a time:
// ds_add_f32 occupies the CU's LDS for 2.9 cycles per active lane (104 for these
// 36 lanes, more than the iteration's vector instructions take), ds_add_f64 for
// 8 cycles in all.  So the accumulators are double where every Gaussian is
// active, and float under an active mask, where few lanes add and the longer
// rounds are worth more.  The sums of a group that does not composite the entry
// are zeros and are not added, unless dL/dcolour is not finite somewhere (0
// times it is NaN): then (`strict`) only groups with a lane in cm are let through.
// `on`: the lanes that may emit.
__device__ __forceinline__ uint64_t rows_of(uint64_t lanes) {  // all lanes of the rows that have one
  constexpr uint64_t kRow = 0x0001000100010001ull;
  lanes |= (lanes >> 8) & 0x00ff00ff00ff00ffull;
  lanes |= (lanes >> 4) & 0x000f000f000f000full;
  lanes |= (lanes >> 2) & 0x0003000300030003ull;
  lanes = (lanes | (lanes >> 1)) & kRow;
  return (lanes << 16) - lanes;
}
template <bool DET, typename Acc>
__device__ __forceinline__ void emit_partial(Acc* s_acc, float* __restrict__ part, uint32_t* __restrict__ pmask,
                                             uint32_t k, uint32_t base, int g16, int slot, uint64_t on, float val) {
  if (!__builtin_amdgcn_inverse_ballot_w64(on)) return;
  if (DET) {
    const uint32_t j = base + k;
    part[((int64_t)j * 16 + g16) * kG2d + slot] = val;
    if (slot == 8) atomicOr(pmask + j, 1u << g16);
  } else if (val != 0.f) {
    atomicAdd(s_acc + (uint32_t)__umul24(k, (uint32_t)kG2d) + slot, (Acc)val);
  }
}

// Same lane layout and group streams as the forward, walking rounds and
// entries back to front from the largest `last` of the workgroup.  Per pixel:
// restore the transmittance in front of the Gaussian (T /= 1 - alpha), form
// dL/dalpha from the colour composited behind it, and add the Gaussian's own
// weighted colour to that suffix.  Entries of
// inactive Gaussians update the per-pixel state but emit no gradient.  The
// nine sums of a group's entry are formed over its 16 lanes in registers and
// added by nine of its lanes to the entry's accumulators in LDS; after each
// round the workgroup adds them, converted, to the records' 2D gradients.
// One global atomic per (entry, workgroup) and component instead of one per
// (entry, group): float atomics are carried out at the memory side (at most
// ~17 G requests/s), which bounded the kernel where most entries are active
// (1M Gaussians, 16 views, 17.3M pixels, all active: 169M -> 31M requests).
// Now bound by the vector instructions of the walk.  Measured there, against
// partials summed straight into the 2D gradients: 9.31 -> 3.89 ms; 500k
// Gaussians at 1245x825 395 -> 279 us, 3M at 1920x1080 with a quarter of them
// active 628 -> 550 us; one list of 4,000 entries, where the walk's latency is
// all, 434 -> 410 us.  What the gradients of needles do not allow (a scalar
// suffix, a shorter tree, the conic applied to the sums: row_sum9,
// alpha_gradient, g2d_component) made 3.69 ms, 225 us and 490 us of 4.33, 298
// and 556, measured before the record indices were read once per round.
template <bool MASKED, bool DET>
__global__ __launch_bounds__(kBlock) void k_render_bwd(const float* __restrict__ rec, const int32_t* __restrict__ bin,
                                                       const uint32_t* __restrict__ vals,
                                                       const uint32_t* __restrict__ ranges,
                                                       const uint32_t* __restrict__ order, int32_t nsplit, int64_t n,
                                                       const float* __restrict__ t_final,
                                                       const uint32_t* __restrict__ last,
                                                       const float* __restrict__ dldc,
                                                       const uint8_t* __restrict__ active, float* __restrict__ g2d,
                                                       float* __restrict__ part, uint32_t* __restrict__ pmask,
                                                       KOpts op, ViewSet vs) {
  constexpr int kBatch = kBwdBatch<MASKED, DET>;
  using Acc = std::conditional_t<MASKED, float, double>;
  __shared__ float4 s_r0[kBatch], s_r1[kBatch], s_r2[kBatch];
  __shared__ RoundLds<kBatch, true> s_round;
  // the staged entries' sums over the workgroup; all zero at the start of a round
  __shared__ Acc s_acc[DET ? 1 : kBatch * kG2d];
  __shared__ alignas(4) uint8_t s_stream[kWaves][kGroups][kBatch];
  __shared__ uint32_t s_last[kWaves * kGroups];  // largest `last` of each group
  const WorkItem wi = work_item(order, ranges, nsplit, vs.tiles_total, false);
  if (wi.skip) return;
  const int32_t tile = wi.tile;
  const int32_t v = view_of_tile(vs, tile);
  const KView& cam = vs.v[v];
  const int32_t lt = tile - cam.tile_base;
  const int32_t tx = lt % cam.tiles_x, ty = lt / cam.tiles_x;
  const int wv = (int)uniform_u32(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int grp = lane >> 4;
  const bool rp = wi.quarter >= 0;  // split work item: rows are consecutive entries
  const LanePixel lp = lane_pixel(tx, ty, wi.quarter, wv, lane, rp);
  const int32_t sx0 = lp.sx0, sy0 = lp.sy0, px = lp.px, py = lp.py;
  const bool inside = lp.on && px < cam.width && py < cam.height;
  const float pxc = (float)px + 0.5f, pyc = (float)py + 0.5f;
  const uint32_t start = uload(ranges + 2 * tile), end = uload(ranges + 2 * tile + 1);
  const int64_t vbase = (int64_t)v * n;
  const int64_t nrec = (int64_t)vs.count * n;
  // the row's 4x4 group among the tile's sixteen (8x8 quarter, then 4x4 group
  // inside it), the same pixels whether or not the tile is split
  const int g16 = rp ? wi.quarter * 4 + wv : wv * 4 + grp;
  set_wave_priority(end - start);
  const int64_t P = vs.pixels_total;
  const int64_t gp = cam.pixel_base + (int64_t)py * cam.width + px;
  float T = 1.f, g[3] = {0.f, 0.f, 0.f};
  uint32_t lst = 0;
  if (inside) {
    T = t_final[gp];
    lst = last[gp];
    for (int k = 0; k < 3; ++k) g[k] = dldc[k * P + gp];
  }
  lst = lst < end - start ? lst : end - start;  // `last` never exceeds the tile's list
  float S[3] = {T * op.bg[0], T * op.bg[1], T * op.bg[2]};  // colour composited behind
  const int slot = sum_slot(lane);  // the sum this lane emits after row_sum9, or -1
  const ChannelPixels gm = channel_pixels(g[0], g[1], g[2], lane);
  const uint64_t emitters = __builtin_amdgcn_ballot_w64(slot >= 0);
  const bool strict = __builtin_amdgcn_ballot_w64(!(fabsf(g[0]) < INFINITY && fabsf(g[1]) < INFINITY &&
                                                    fabsf(g[2]) < INFINITY)) != 0;
  {
    uint32_t m = lst;  // over the 16 lanes of a group; split rows hold the same pixels
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) {
      const uint32_t y = __shfl_xor(m, o, kWave);
      m = y > m ? y : m;
    }
    if ((lane & 15) == 0) s_last[wv * kGroups + grp] = m;
  }
  __syncthreads();
  uint32_t bjmax = 0;
#pragma unroll
  for (int k = 0; k < kWaves * kGroups; ++k) bjmax = s_last[k] > bjmax ? s_last[k] : bjmax;
  bjmax = uniform_u32(bjmax);
  if (bjmax == 0u) return;
  if (!DET) {
    const int slots = bjmax < (uint32_t)kBatch ? (int)bjmax : kBatch;  // no round is longer
    for (int q = threadIdx.x; q < slots * kG2d; q += kBlock) s_acc[q] = Acc(0);
  }
  const int32_t ix0 = tx * kTile + (rp ? (wi.quarter & 1) * 8 : 0), iy0 = ty * kTile + (rp ? (wi.quarter >> 1) * 8 : 0);
  // Rounds cover [base, top) downwards from start + bjmax.  Staging pipeline:
  // the records of the next round and the list indices of the one after are
  // in flight while a round is processed.
  // In a split work item which entries share a product of transmittances, and
  // with it the rounding, must not depend on the rounds' length: fours are of one
  // chunk of 64, and the chunks are those of rounds of 256 (the last `tail`
  // entries counted from the start, the others from the end).
  const uint32_t tail = bjmax > 0u ? ((bjmax - 1u) & 255u) + 1u : 0u;
  auto round_base = [&](uint32_t top) {
    const uint32_t r = top - start;
    if (kBatch < 256 && rp) {
      if (r > tail) return r - tail > (uint32_t)kBatch ? top - kBatch : start + tail;
      return r > (uint32_t)kBatch ? start + kBatch : start;
    }
    return r > (uint32_t)kBatch ? top - kBatch : start;
  };
  uint32_t top = start + bjmax;
  uint32_t base = round_base(top);
  const uint32_t mine_at = threadIdx.x;
  const bool stager = mine_at < (uint32_t)kBatch;
  StagedB cur = fetch_entry_bwd<MASKED>(rec, bin, active, stager && base + mine_at < top ? vals[base + mine_at] : 0u,
                                        stager && base + mine_at < top, nrec, vbase);
  uint32_t nbase = round_base(base), ntop = base;
  uint32_t nidx = stager && nbase + mine_at < ntop ? vals[nbase + mine_at] : 0u;
  while (top > start) {
    const uint32_t count = top - base;
    // pixels whose last entry lies above the round's, and each chunk's, first
    const uint64_t am = __builtin_amdgcn_ballot_w64(lst > base - start);
#pragma unroll
    for (int c = 0; c < kBatch / kWave; ++c) {
      const uint64_t in = c == 0 ? am : __builtin_amdgcn_ballot_w64(lst > base - start + c * kWave);
      if (lane == 0) s_round.active[wv][c] = in;
    }
    __syncthreads();  // the previous round's entries are consumed
    if (stager) {
      s_r0[mine_at] = cur.r0;
      s_r1[mine_at] = cur.r1;
      s_r2[mine_at] = cur.r2;
    }
    uint64_t walked = test_round(s_round, s_last, base + mine_at - start, rp, ix0, iy0, cur.box, cur.r0, cur.r1,
                                 stager && mine_at < count, wv, fresh(lane), op.log2_alpha_min);
    if (MASKED) walked &= __builtin_amdgcn_ballot_w64(cur.r2.w > 0.f);
    __syncthreads();
    {
      // next round [nbase, ntop) and the one after it
      cur = fetch_entry_bwd<MASKED>(rec, bin, active, nidx, stager && ntop > start && nbase + mine_at < ntop, nrec,
                                    vbase);
      const uint32_t nnbase = round_base(nbase);
      nidx = (stager && nbase > start && nnbase + mine_at < nbase) ? vals[nnbase + mine_at] : 0u;
    }
    if (am != 0) {
      int n4[kGroups];
      make_streams<false>(s_round, s_stream[wv], 1, rp, rp, wv, fresh(lane), n4);
      // round-relative offset from which on the pixel composited nothing
      const uint32_t lim = round_limit(lst, base - start, kBatch);
      // Split work item: row r takes the r-th latest of the next four entries
      // of the group's stream.  The transmittance in front of each is the
      // product of 1 / (1 - alpha) over the rows up to it, its suffix colour
      // the sum of the weighted colours of the rows before it; the nine
      // partials of each row's entry are then summed over the row as usual.
      int left = rp ? n4[kBatch / kWave - 1] : 0;
      auto chunk_first = [&](int at) { return at > n4[2] ? n4[2] : at > n4[1] ? n4[1] : at > n4[0] ? n4[0] : 0; };
      int floor = chunk_first(left);
      uint32_t offn = s_stream[wv][0][left - floor > grp ? left - 1 - grp : floor];
      while (left > 0) {
        const bool hr = left - floor > grp;
        const uint32_t off = offn * 16u;
        left = left - floor > kGroups ? left - kGroups : floor;
        floor = chunk_first(left);
        offn = s_stream[wv][0][left - floor > grp ? left - 1 - grp : floor];
        const bool val = hr && off < lim;
        const float4 r0 = lds_at(s_r0, off), r1 = lds_at(s_r1, off), c4 = lds_at(s_r2, off);
        const float dx = (pxc - r0.x) - r0.z, dy = (pyc - r0.y) - r0.w;
        const float ee = r1.w - (r1.x * dx * dx + r1.y * dx * dy + r1.z * dy * dy);
        const float G2 = __builtin_amdgcn_exp2f(ee);
        const bool inc = val && ee >= op.log2_alpha_min;
        const bool act = MASKED ? inc && c4.w > 0.f : inc;
        const float al = fminf(op.alpha_max, G2);
        const float iom = __builtin_amdgcn_rcpf(1.f - al);
        const RowScan tr = rows_scan_mul(inc ? iom : 1.f, grp);
        const float Tr = T * tr.incl;
        const float wgt = inc ? al * Tr : 0.f;
        const RowScan u0 = rows_scan_add(wgt * c4.x, grp), u1 = rows_scan_add(wgt * c4.y, grp),
                      u2 = rows_scan_add(wgt * c4.z, grp);
        const float Sr[3] = {S[0] + u0.excl, S[1] + u1.excl, S[2] + u2.excl};
        const float ga = alpha_gradient(g, c4, Tr, iom, Sr);
        float pv[6];
        const float wa = !MASKED || act ? wgt : 0.f;
        const float gal = (act && G2 < op.alpha_max) ? ga * al : 0.f;
        pv[5] = gal;
        const float gx = gal * dx, gy = gal * dy;
        pv[0] = gal * __builtin_fmaf(2.f, r1.x * dx, r1.y * dy);
        pv[1] = gal * __builtin_fmaf(2.f, r1.z * dy, r1.y * dx);
        pv[2] = gx * dx;
        pv[3] = gx * dy;
        pv[4] = gy * dy;
        T = T * tr.total;
        S[0] += u0.total;
        S[1] += u1.total;
        S[2] += u2.total;
        // (a weight is positive wherever the entry is composited)
        const uint64_t cm = __builtin_amdgcn_ballot_w64(wa > 0.f);
        if (cm == 0) continue;
        uint64_t on = emitters;
        if (DET || strict) on &= rows_of(cm);
        emit_partial<DET>(s_acc, part, pmask, off >> 4, base, g16, slot, on, row_sum9(pv, wa, gm, lane));
      }
      // One entry of the group's stream per iteration, latest first; the
      // transmittance is restored through them in reverse order.
      const int mine = grp == 0 ? n4[0] : grp == 1 ? n4[1] : grp == 2 ? n4[2] : n4[3];
      const int longest = (int)uniform_u32((uint32_t)(rp ? 0 : max4(n4)));
      const uint8_t* sp = &s_stream[wv][grp][0] + (mine > 0 ? mine - 1 : 0);
      uint32_t ahead = *sp;
      for (int i = 0; i < longest; ++i) {
        const uint32_t k = (uint32_t)fresh((int)ahead), at = k * 16u;
        const bool val = i < mine && at < lim;
        sp -= i + 1 < mine ? 1 : 0;
        ahead = *sp;
        const float4 r0 = lds_at(s_r0, at), r1 = lds_at(s_r1, at), c4 = lds_at(s_r2, at);
        const float dx = (pxc - r0.x) - r0.z, dy = (pyc - r0.y) - r0.w;
        const float ee = r1.w - (r1.x * dx * dx + r1.y * dx * dy + r1.z * dy * dy);
        const float G2 = __builtin_amdgcn_exp2f(ee);
        // Branch-free per lane: a lane that skips the entry multiplies its
        // partials by zero and keeps its transmittance; staged records are
        // finite, so the zero products are zeros.  Transmittance in front of
        // the entry, its partials, then its colour joins the suffix.
        const bool inc = val && ee >= op.log2_alpha_min;
        const bool act = MASKED ? inc && c4.w > 0.f : inc;
        const float al = fminf(op.alpha_max, G2);
        const float iom = __builtin_amdgcn_rcpf(1.f - al);
        T = inc ? T * iom : T;
        const float wgt = inc ? al * T : 0.f;
        const float ga = alpha_gradient(g, c4, T, iom, S);
        S[0] = __builtin_fmaf(wgt, c4.x, S[0]);
        S[1] = __builtin_fmaf(wgt, c4.y, S[1]);
        S[2] = __builtin_fmaf(wgt, c4.z, S[2]);
        const float wa = !MASKED || act ? wgt : 0.f;
        const uint64_t cm = __builtin_amdgcn_ballot_w64(wa > 0.f);
        if (cm == 0) continue;
        uint64_t on = emitters;
        if (DET || strict) on &= rows_of(cm);
        float pv[6];
        // the clamped alpha has no gradient with respect to opacity or shape
        const float gal = (act && G2 < op.alpha_max) ? ga * al : 0.f;
        pv[5] = gal;
        const float gx = gal * dx, gy = gal * dy;
        pv[0] = gal * __builtin_fmaf(2.f, r1.x * dx, r1.y * dy);
        pv[1] = gal * __builtin_fmaf(2.f, r1.z * dy, r1.y * dx);
        pv[2] = gx * dx;
        pv[3] = gx * dy;
        pv[4] = gy * dy;
        emit_partial<DET>(s_acc, part, pmask, k, base, g16, slot, on, row_sum9(pv, wa, gm, lane));
      }
    }
    if (!DET) {
      // Wave w adds the walked active entries of chunk w, which it tested, to
      // their records: seven entries of nine consecutive components at a time,
      // so an entry's adds leave in one or two requests.  It clears what it
      // has read.  The record indices are read again once for the chunk, while
      // the wave waits for the others: a read per turn of the loop had its
      // latency in every one (4.00 -> 3.87 ms there, 454 -> 410 us on the one
      // list).
      const int fl = fresh(lane);
      const bool mine = __builtin_amdgcn_inverse_ballot_w64(walked);  // (its index is valid)
      const uint32_t who = mine ? vals[base + wv * kWave + fl] : 0u;
      __syncthreads();
      const int fe = fl / kG2d, fc = fl - fe * kG2d;
      const int cnt = (int)__popcll(walked);
      uint8_t* list = &s_stream[wv][0][0];  // this wave's streams are walked
      AliasedU32* records = reinterpret_cast<AliasedU32*>(list + kWave);
      static_assert(kWave * 5 <= kGroups * kBatch, "slot and record of a chunk's entries");
      if (mine) {
        const uint32_t at =
            __builtin_amdgcn_mbcnt_hi((uint32_t)(walked >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)walked, 0u));
        list[at] = (uint8_t)(wv * kWave + fl);
        records[at] = who;
      }
      wave_sync();
#pragma unroll 1
      for (int e = fe < kWave / kG2d ? fe : kWave; e < cnt; e += kWave / kG2d) {
        const uint32_t k = list[e];
        const uint32_t r = records[e];
        Acc* ap = s_acc + k * kG2d;
        const float val = g2d_component(fc, (float)ap[fc], fabsf(s_r2[k].w));
        ap[fc] = Acc(0);
        if (val != 0.f) atomicAdd(g2d + (int64_t)r * kG2d + fc, val);
      }
    }
    top = base;
    base = nbase;
    nbase = round_base(nbase);
    ntop = base;
  }
}

__global__ void k_zero_f32(float* __restrict__ p, int64_t count) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (; i < count; i += stride) p[i] = 0.f;
}

// Deterministic gradient reduction.  Step 1, one workgroup per tile: for each
// entry of the tile's list, the sum of the sixteen groups' slots in group
// order, stored at the pair's emission index e = offsets[r] + the tile's rank
// among the tiles the record was emitted for (row-major over its box, only the
// kept tiles under tile culling), so every record's pairs sit side by side.
__global__ __launch_bounds__(kBlock) void k_det_tile(const uint32_t* __restrict__ vals,
                                                     const uint32_t* __restrict__ ranges,
                                                     const int32_t* __restrict__ bin, const float* __restrict__ rec,
                                                     float tile_cull, const uint32_t* __restrict__ offsets,
                                                     const float* __restrict__ part,
                                                     const uint32_t* __restrict__ pmask, float* __restrict__ tpart,
                                                     int64_t nrec, int64_t n_isect, ViewSet vs) {
  const int32_t tile = (int32_t)blockIdx.x;
  const int32_t v = view_of_tile(vs, tile);
  const int32_t lt = tile - vs.v[v].tile_base;
  const int32_t tx = lt % vs.v[v].tiles_x, ty = lt / vs.v[v].tiles_x;
  const uint32_t start = ranges[2 * tile], end = ranges[2 * tile + 1];
  for (uint32_t j = start + threadIdx.x; j < end; j += kBlock) {
    const uint32_t r = vals[j];
    if ((int64_t)r >= nrec) continue;
    const int4 b = reinterpret_cast<const int4*>(bin)[r];
    const int32_t x0 = b.x & 0xffff, x1 = (int32_t)((uint32_t)b.x >> 16);
    const int32_t y0 = b.y & 0xffff, y1 = (int32_t)((uint32_t)b.y >> 16);
    const int32_t tx0 = x0 >> 4, tx1 = x1 >> 4, ty0 = y0 >> 4;
    uint32_t k;
    if (b.w < (tx1 - tx0 + 1) * ((y1 >> 4) - ty0 + 1)) {
      // tile culling emitted only the kept tiles: rank among those
      const float4* R4 = reinterpret_cast<const float4*>(rec + (int64_t)r * kRecFloats);
      const float4 r0 = R4[0], r1 = R4[1];
      k = 0;
      for (int32_t yy = ty0; yy <= ty; ++yy)
        for (int32_t xx = tx0; xx <= tx1 && (yy < ty || xx < tx); ++xx)
          k += tile_kept(r0, r1, xx, yy, x0, x1, y0, y1, tile_cull) ? 1u : 0u;
    } else {
      k = (uint32_t)((ty - ty0) * (tx1 - tx0 + 1) + (tx - tx0));
    }
    const int64_t e = (int64_t)offsets[r] + k;
    if (e >= n_isect) continue;
    float acc[kG2d];
#pragma unroll
    for (int c = 0; c < kG2d; ++c) acc[c] = 0.f;
    for (uint32_t m = pmask[j]; m != 0u; m &= m - 1u) {
      const float* sp = part + ((int64_t)j * 16 + (__builtin_ctz(m))) * kG2d;
#pragma unroll
      for (int c = 0; c < kG2d; ++c) acc[c] += sp[c];
    }
#pragma unroll
    for (int c = 0; c < kG2d; ++c) tpart[e * kG2d + c] = acc[c];
  }
}

// Step 2, one thread per record: its pairs' sums in emission order (tiles of
// its box row-major), converted to the record's 2D gradient and added to it.
__global__ __launch_bounds__(kBlock) void k_det_record(const int32_t* __restrict__ bin, const float* __restrict__ rec,
                                                       const uint32_t* __restrict__ offsets,
                                                       const float* __restrict__ tpart, float* __restrict__ g2d,
                                                       int64_t nrec, int64_t n_isect) {
  const int64_t r = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (r >= nrec) return;
  const int32_t tt = bin[4 * r + 3];
  if (tt <= 0) return;
  const int64_t e0 = offsets[r];
  if (e0 + tt > n_isect) return;
  float acc[kG2d];
#pragma unroll
  for (int c = 0; c < kG2d; ++c) acc[c] = 0.f;
  for (int32_t k = 0; k < tt; ++k) {
#pragma unroll
    for (int c = 0; c < kG2d; ++c) acc[c] += tpart[(e0 + k) * kG2d + c];
  }
  const float op = rec[r * kRecFloats + 11];
#pragma unroll
  for (int c = 0; c < kG2d; ++c) g2d[r * kG2d + c] += g2d_component(c, acc[c], op);
}

size_t det_ws_bytes(int64_t n_isect) {
  const int64_t ni = n_isect > 0 ? n_isect : 1;
  return align256((size_t)ni * 4) + align256((size_t)ni * 16 * kG2d * 4) + align256((size_t)ni * kG2d * 4);
}

template <bool ACC, bool OUT>
static void launch_fwd(int depth_mode, dim3 grid, hipStream_t s, const gs_projected_t* proj, const uint32_t* vals,
                       const uint32_t* ranges, const uint32_t* order, int64_t n, const gs_scene_t* scene, const FwdOut& o, const KOpts& op,
                       int32_t per_view, const ViewSet& vs) {
  const float* m = scene ? scene->means : nullptr;
  const float* sc = scene ? scene->scales : nullptr;
  const float* q = scene ? scene->quats : nullptr;
  if (depth_mode == GS_DEPTH_CENTER)
    hipLaunchKernelGGL((k_render_fwd<ACC, OUT, GS_DEPTH_CENTER>), grid, dim3(kBlock), 0, s, proj->rec, proj->bin, vals,
                       ranges, order, split_tiles(order, vs.tiles_total), n, m, sc, q, o, op, per_view, vs);
  else if (depth_mode == GS_DEPTH_BLEND)
    hipLaunchKernelGGL((k_render_fwd<ACC, OUT, GS_DEPTH_BLEND>), grid, dim3(kBlock), 0, s, proj->rec, proj->bin, vals,
                       ranges, order, split_tiles(order, vs.tiles_total), n, m, sc, q, o, op, per_view, vs);
  else
    hipLaunchKernelGGL((k_render_fwd<ACC, OUT, GS_DEPTH_MID>), grid, dim3(kBlock), 0, s, proj->rec, proj->bin, vals,
                       ranges, order, split_tiles(order, vs.tiles_total), n, m, sc, q, o, op, per_view, vs);
}

}  // namespace msplat

using namespace msplat;

extern "C" {

int32_t gs_render_forward(const gs_scene_t* scene, const gs_projected_t* proj, const uint32_t* vals,
                          const uint32_t* ranges, const uint32_t* tile_order, const gs_camera_t* cams, int32_t V,
                          const gs_opts_t* opts, const gs_fwd_out_t* out, const gs_accum_t* acc, void* stream) {
  int32_t st = check_scene(scene);
  if (st != GS_OK) return st;
  if (!proj || !opts || !out || !ranges) { set_error("proj/opts/out/ranges NULL"); return GS_ERR_NULL; }
  if (opts->depth_mode < 0 || opts->depth_mode > 2) { set_error("depth_mode"); return GS_ERR_UNSUPPORTED; }
  ViewSet vs;
  if ((st = build_views(cams, V, &vs)) != GS_OK) return st;
  if ((st = check_records(V, scene->n)) != GS_OK) return st;
  if (!out->color || !out->t_final || !out->last || !out->imax) { set_error("forward output NULL"); return GS_ERR_NULL; }
  const bool accum = (opts->flags & GS_ACCUM_IMPORTANCE) != 0;
  if (accum && !acc) { set_error("GS_ACCUM_IMPORTANCE without accumulators"); return GS_ERR_NULL; }
  if (scene->n > 0 && (!proj->rec || !proj->bin)) { set_error("projected buffers NULL"); return GS_ERR_NULL; }
  FwdOut o{out->color, out->depth, out->imax, out->t_final, out->last, out->n_contrib, out->hit,
           accum ? acc->importance : nullptr, accum ? acc->wmax : nullptr, accum ? acc->area : nullptr};
  const KOpts op = make_kopts(opts);
  const int32_t per_view = (opts->flags & GS_ACCUM_PER_VIEW) ? 1 : 0;
  dim3 grid(vs.tiles_total + 3 * split_tiles(tile_order, vs.tiles_total));
  hipStream_t s = (hipStream_t)stream;
  if (accum)
    launch_fwd<true, true>(opts->depth_mode, grid, s, proj, vals, ranges, tile_order, scene->n, scene, o, op, per_view,
                           vs);
  else
    launch_fwd<false, true>(opts->depth_mode, grid, s, proj, vals, ranges, tile_order, scene->n, scene, o, op,
                            per_view, vs);
  MS_CHECK_LAUNCH("render_forward");
  return GS_OK;
}

int32_t gs_accumulate_importance(const gs_projected_t* proj, const uint32_t* vals, const uint32_t* ranges,
                                 const uint32_t* tile_order, const gs_camera_t* cams, int32_t V, int64_t n,
                                 const gs_opts_t* opts, const gs_accum_t* acc, void* stream) {
  if (!proj || !opts || !acc || !ranges) { set_error("proj/opts/acc/ranges NULL"); return GS_ERR_NULL; }
  if (n < 0) { set_error("n < 0"); return GS_ERR_SHAPE; }
  ViewSet vs;
  int32_t st = build_views(cams, V, &vs);
  if (st != GS_OK) return st;
  if ((st = check_records(V, n)) != GS_OK) return st;
  if (n > 0 && (!proj->rec || !proj->bin)) { set_error("projected buffers NULL"); return GS_ERR_NULL; }
  FwdOut o{};
  o.imp = acc->importance;
  o.wmax = acc->wmax;
  o.area = acc->area;
  const KOpts op = make_kopts(opts);
  const int32_t per_view = (opts->flags & GS_ACCUM_PER_VIEW) ? 1 : 0;
  hipLaunchKernelGGL((k_render_fwd<true, false, GS_DEPTH_CENTER>),
                     dim3(vs.tiles_total + 3 * split_tiles(tile_order, vs.tiles_total)), dim3(kBlock), 0,
                     (hipStream_t)stream, proj->rec, proj->bin, vals, ranges, tile_order,
                     split_tiles(tile_order, vs.tiles_total), n, nullptr, nullptr, nullptr,
                     o, op, per_view, vs);
  MS_CHECK_LAUNCH("accumulate_importance");
  return GS_OK;
}

int32_t gs_render_backward_pixels(const gs_projected_t* proj, const uint32_t* vals, const uint32_t* ranges,
                                  const uint32_t* tile_order, const gs_camera_t* cams, int32_t V, int64_t n,
                                  const gs_opts_t* opts, const float* t_final, const uint32_t* last,
                                  const float* dl_dcolor, const uint8_t* active, float* grad2d, void* stream) {
  if (!proj || !opts || !ranges || !t_final || !last || !dl_dcolor) { set_error("argument NULL"); return GS_ERR_NULL; }
  if (n < 0) { set_error("n < 0"); return GS_ERR_SHAPE; }
  ViewSet vs;
  int32_t st = build_views(cams, V, &vs);
  if (st != GS_OK) return st;
  if ((st = check_records(V, n)) != GS_OK) return st;
  if (n == 0) return GS_OK;
  if (!proj->rec || !proj->bin || !grad2d) { set_error("buffer NULL"); return GS_ERR_NULL; }
  const KOpts op = make_kopts(opts);
  hipStream_t s = (hipStream_t)stream;
  const dim3 grid(vs.tiles_total + 3 * split_tiles(tile_order, vs.tiles_total));
  if (active)
    hipLaunchKernelGGL((k_render_bwd<true, false>), grid, dim3(kBlock), 0, s, proj->rec, proj->bin, vals,
                       ranges, tile_order, split_tiles(tile_order, vs.tiles_total), n, t_final, last, dl_dcolor,
                       active, grad2d, nullptr, nullptr, op, vs);
  else
    hipLaunchKernelGGL((k_render_bwd<false, false>), grid, dim3(kBlock), 0, s, proj->rec, proj->bin, vals,
                       ranges, tile_order, split_tiles(tile_order, vs.tiles_total), n, t_final, last, dl_dcolor,
                       active, grad2d, nullptr, nullptr, op, vs);
  MS_CHECK_LAUNCH("render_backward_pixels");
  return GS_OK;
}

size_t gs_render_backward_det_workspace_size(int64_t n_isect) { return det_ws_bytes(n_isect); }

int32_t gs_render_backward_pixels_det(const gs_projected_t* proj, const uint32_t* vals, const uint32_t* ranges,
                                      const uint32_t* tile_order, const uint32_t* offsets, const gs_camera_t* cams,
                                      int32_t V, int64_t n, int64_t n_isect, const gs_opts_t* opts,
                                      const float* t_final, const uint32_t* last, const float* dl_dcolor,
                                      const uint8_t* active, float* grad2d, void* ws, size_t ws_bytes,
                                      void* stream) {
  if (!proj || !opts || !ranges || !t_final || !last || !dl_dcolor) { set_error("argument NULL"); return GS_ERR_NULL; }
  if (n < 0 || n_isect < 0) { set_error("n < 0 or n_isect < 0"); return GS_ERR_SHAPE; }
  ViewSet vs;
  int32_t st = build_views(cams, V, &vs);
  if (st != GS_OK) return st;
  if ((st = check_records(V, n)) != GS_OK) return st;
  if (n == 0 || n_isect == 0) return GS_OK;
  if (!proj->rec || !proj->bin || !grad2d || !vals || !offsets || !ws) { set_error("buffer NULL"); return GS_ERR_NULL; }
  if (n_isect >= (int64_t(1) << 32)) { set_error("n_isect of 2^32 or more"); return GS_ERR_CAPACITY; }
  if (ws_bytes < det_ws_bytes(n_isect)) { set_error("deterministic backward workspace too small"); return GS_ERR_CAPACITY; }
  char* p = (char*)ws;
  uint32_t* pmask = (uint32_t*)p; p += align256((size_t)n_isect * 4);
  float* part = (float*)p; p += align256((size_t)n_isect * 16 * kG2d * 4);
  float* tpart = (float*)p;
  const KOpts op = make_kopts(opts);
  hipStream_t s = (hipStream_t)stream;
  if ((st = launch_fill(pmask, 0u, n_isect, s)) != GS_OK) return st;
  const dim3 grid(vs.tiles_total + 3 * split_tiles(tile_order, vs.tiles_total));
  if (active)
    hipLaunchKernelGGL((k_render_bwd<true, true>), grid, dim3(kBlock), 0, s, proj->rec, proj->bin, vals,
                       ranges, tile_order, split_tiles(tile_order, vs.tiles_total), n, t_final, last, dl_dcolor,
                       active, grad2d, part, pmask, op, vs);
  else
    hipLaunchKernelGGL((k_render_bwd<false, true>), grid, dim3(kBlock), 0, s, proj->rec, proj->bin, vals,
                       ranges, tile_order, split_tiles(tile_order, vs.tiles_total), n, t_final, last, dl_dcolor,
                       active, grad2d, part, pmask, op, vs);
  MS_CHECK_LAUNCH("render_backward_pixels_det");
  const int64_t nrec = (int64_t)V * n;
  hipLaunchKernelGGL(k_det_tile, dim3((unsigned)vs.tiles_total), dim3(kBlock), 0, s, vals, ranges, proj->bin,
                     proj->rec, proj->tile_cull_log2_alpha, offsets, part, pmask, tpart, nrec, n_isect, vs);
  hipLaunchKernelGGL(k_det_record, dim3(grid_1d(nrec)), dim3(kBlock), 0, s, proj->bin, proj->rec, offsets, tpart,
                     grad2d, nrec, n_isect);
  MS_CHECK_LAUNCH("deterministic reduction");
  return GS_OK;
}

int32_t gs_render_backward(const gs_scene_t* scene, const gs_projected_t* proj, const uint32_t* vals,
                           const uint32_t* ranges, const uint32_t* tile_order, const gs_camera_t* cams, int32_t V,
                           const gs_opts_t* opts, const float* t_final, const uint32_t* last,
                           const float* dl_dcolor, const uint8_t* active, float* grad2d, const gs_grads_t* grads,
                           void* stream) {
  int32_t st = check_scene(scene);
  if (st != GS_OK) return st;
  if (scene->n > 0) {
    if (!grad2d) { set_error("grad2d NULL"); return GS_ERR_NULL; }
    const int64_t count = (int64_t)V * scene->n * kG2d;
    int64_t blocks = (count + kBlock - 1) / kBlock;
    if (blocks > 16384) blocks = 16384;
    if (V >= 1 && V <= GS_MAX_VIEWS) {
      hipLaunchKernelGGL(k_zero_f32, dim3((unsigned)blocks), dim3(kBlock), 0, (hipStream_t)stream, grad2d, count);
      MS_CHECK_LAUNCH("zero grad2d");
    }
  }
  st = gs_render_backward_pixels(proj, vals, ranges, tile_order, cams, V, scene->n, opts, t_final, last, dl_dcolor,
                                 active, grad2d, stream);
  if (st != GS_OK) return st;
  return gs_project_backward(scene, proj, cams, V, opts, grad2d, active, grads, stream);
}

}  // extern "C"
