// matrix.hip -- IoU matrices (one block a.count x b.count, or ragged segments
// such as per-scene self-pairs of 3D boxes, Sec. IV-A case study at scale) and
// their backward from the saved per-pair state (Sec. II-B: nx and xflags).
//
// The forward is split by register pressure into lean cull and list kernels
// and one dense exact kernel, with no shared counter anywhere:
//   k_matrix_cull -- survivor masks and counts per tile of R rows x 2048 / R
//     columns of one segment (R = 4, 8 or 16, chosen per call).  A lane holds a
//     row; the pairs it tests are those whose bins on every axis overlap, found
//     64 columns at a time from bit sets in LDS (all 64 where those are many).
//   k_matrix_list -- lays the work list out tile by tile, deterministically
//     (the prefix of the tile counts, then the masks' survivors), while its
//     other workgroups write the output's zeros as a flat stream.
//   k_matrix_exact -- one lane per survivor with every lane busy: the exact
//     pair forward, the IoU written to its place in the output, nx / xflags
//     kept in the work list for the backward; and the self diagonal's 1s.
// (k_scan_totals sums chunks of tile counts first where the table is too
// large for each list workgroup to sum the counts before its own.)
// c5 (64 scenes, 93.6 M pairs) takes 23 + 63 + 35 us; a kernel that tested every
// pair and wrote the tiles' values (103 us), two scan passes (11), a fill of
// the list (13) and the exact pass (31) took 162 with the segments' prefixes.
// Grids walk the units or tiles of all segments, whose sizes are on the
// device (the prefixes over segments are computed there, so everything is
// graph-capturable).  The backward (k_matrix_bwd) gives one wavefront a row
// group of 8 rows, whatever the tile shape: the entries of the tile rows
// that cover it are one contiguous range of the work list; each step's row
// gradients are summed without atomics (sorted by row in LDS, each lane
// adding up one (row, vertex) run in a fixed order) and every row is written
// once.  Self pairs need nothing else: entries (i, k) and (k, i) are one
// unordered pair evaluated with the lower index first, so the row role of either entry is that pair's
// gradient for the row's box, weighted by both entries' upstream gradients;
// for two different sets the column gradients are added with global atomics, a
// row's floats on consecutive lanes.  A single block of few or wide row groups
// gives each a workgroup, whose wavefronts take its steps in turn.
#include <algorithm>
#include <mutex>
#include <type_traits>
#include <utility>

#include "geom.hpp"
#include "internal.hpp"

namespace dgal {

constexpr int kTilePairs = DGAL_TILE_PAIRS;
constexpr int kCullBlock = 256;   // four independent wavefronts
constexpr int kScanBlock = 1024;
constexpr int kListBlock = 256;
constexpr int kListTiles = kListBlock;  // tiles of a list step
constexpr int kFillSegBlocks = 2048;    // workgroups that fill blocks with gaps between them
// tables of up to this many tiles are summed by the list pass itself
constexpr int64_t kListDirect = 65536;
constexpr int kExactBlock = 256;
constexpr int kMaxSeg = DGAL_MAX_SEGMENTS;
static_assert(kTilePairs == 2048, "32 words of survivor bits per tile");

// log2 of a supported tile row count (4, 8, 16), or -1.
inline int tile_rows_log2(int rows) {
  return rows == 4 ? 2 : (rows == 8 ? 3 : (rows == 16 ? 4 : -1));
}

struct Segment {
  int64_t a0, b0, na, nb, out0;
  bool ok;
};

struct SegArgs {
  const int64_t* a_off;  // NULL => one segment
  const int64_t* b_off;
  const int64_t* out_off;
  int nseg;
  int64_t a_count, b_count, out_size;
  int self_pairs;
  const int64_t* tile_prefix;   // [nseg+1] (segmented), from the cull pass or k_seg_prep
  const int64_t* group_prefix;  // [nseg+1] row groups (segmented), likewise
  int rows_log2;                // tiles of 2^rows_log2 rows x 2^(11 - rows_log2) columns
};

__device__ __forceinline__ Segment load_segment(const SegArgs& a, int s) {
  Segment g;
  if (a.a_off == nullptr) {
    g.a0 = 0;
    g.b0 = 0;
    g.na = a.a_count;
    g.nb = a.b_count;
    g.out0 = 0;
    g.ok = true;
    return g;
  }
  const int64_t a0 = a.a_off[s], a1 = a.a_off[s + 1], b0 = a.b_off[s], b1 = a.b_off[s + 1];
  const int64_t o0 = a.out_off[s];
  g.a0 = a0;
  g.b0 = b0;
  g.na = a1 - a0;
  g.nb = b1 - b0;
  g.out0 = o0;
  g.ok = a0 >= 0 && a1 >= a0 && a1 <= a.a_count && b0 >= 0 && b1 >= b0 && b1 <= a.b_count &&
         o0 >= 0 && o0 <= a.out_size && g.nb < (1 << 24) &&
         (g.nb == 0 || g.na <= (a.out_size - o0) / g.nb) &&
         (!a.self_pairs || (a0 == b0 && a1 == b1));
  if (s > 0) {  // blocks are laid out in segment order without overlap
    const int64_t pna = a.a_off[s] - a.a_off[s - 1], pnb = a.b_off[s] - a.b_off[s - 1];
    g.ok = g.ok && o0 >= a.out_off[s - 1] + pna * pnb;
  }
  return g;
}

// Backward row groups, tile rows and tile columns of a segment.
__device__ __forceinline__ int64_t groups_of(const Segment& g) {
  return (g.na > 0 && g.nb > 0) ? (g.na + kGroupRows - 1) / kGroupRows : 0;
}
__device__ __forceinline__ int64_t tile_rows_of(const Segment& g, int rl) {
  return (g.na > 0 && g.nb > 0) ? (g.na + (1 << rl) - 1) >> rl : 0;
}
__device__ __forceinline__ int64_t col_tiles_of(const Segment& g, int rl) {
  const int cl = 11 - rl;
  return (g.nb + (1 << cl) - 1) >> cl;
}

// Tile and row-group prefixes over segments (one workgroup), for a backward
// whose forward did not keep them.  Rejected segments own nothing and raise
// kErrSegment.
__global__ __launch_bounds__(256) void k_seg_prep(SegArgs a, int* err, int64_t* tile_prefix,
                                                  int64_t* group_prefix) {
  __shared__ int64_t part_t[256], part_g[256];
  const int tid = threadIdx.x;
  const int per = (a.nseg + 255) / 256;
  const int s0 = min(a.nseg, tid * per), s1 = min(a.nseg, s0 + per);
  int64_t st = 0, sg = 0;
  for (int s = s0; s < s1; ++s) {
    const Segment g = load_segment(a, s);
    if (!g.ok) {
      raise_error(err, kErrSegment);
      continue;
    }
    sg += groups_of(g);
    st += tile_rows_of(g, a.rows_log2) * col_tiles_of(g, a.rows_log2);
  }
  part_t[tid] = st;
  part_g[tid] = sg;
  __syncthreads();
  for (int d = 1; d < 256; d <<= 1) {  // inclusive scans
    const int64_t vt = tid >= d ? part_t[tid - d] : 0;
    const int64_t vg = tid >= d ? part_g[tid - d] : 0;
    __syncthreads();
    part_t[tid] += vt;
    part_g[tid] += vg;
    __syncthreads();
  }
  int64_t rt = tid > 0 ? part_t[tid - 1] : 0, rg = tid > 0 ? part_g[tid - 1] : 0;
  if (tid == 0) {
    tile_prefix[0] = 0;
    group_prefix[0] = 0;
  }
  for (int s = s0; s < s1; ++s) {
    const Segment g = load_segment(a, s);
    if (g.ok) {
      rg += groups_of(g);
      rt += tile_rows_of(g, a.rows_log2) * col_tiles_of(g, a.rows_log2);
    }
    tile_prefix[s + 1] = rt;
    group_prefix[s + 1] = rg;
  }
}

// Last s with prefix[s] <= v (the segment that owns item v of a prefix).
__device__ __forceinline__ int find_segment(const int64_t* prefix, int nseg, int64_t v) {
  int lo = 0, hi = nseg - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (prefix[mid] <= v) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// The same search by a whole wavefront, for a wave-uniform v: each round
// loads up to 64 evenly spaced entries of the remaining range (one a lane)
// and keeps the span from the last one not past v, so up to 64 segments take
// one round of loads and up to 4096 two (the scalar search above takes a
// dependent load per halving).
__device__ __forceinline__ int wave_find_segment(const int64_t* prefix, int nseg, int64_t v) {
  const int lane = threadIdx.x & 63;
  int lo = 0, hi = nseg;  // the answer lies in [lo, hi)
  while (hi - lo > 1) {
    const int step = (hi - lo + 63) >> 6;
    const int i = lo + lane * step;
    const uint64_t m = __ballot(i < hi && prefix[i] <= v);
    const int k = m != 0ull ? 63 - __clzll(m) : 0;
    lo += k * step;
    hi = min(hi, lo + step);
  }
  return lo;
}

// Axis-aligned bounds and z-extent of one box (padded slots repeat vertex 0,
// so the bounds over all K slots are the polygon's).
struct Bounds {
  float x0, y0, x1, y1, lo, hi;
};

template <int K, bool FIXED, bool Z3>
__device__ __forceinline__ Bounds box_bounds(const PolyArgs& p, int64_t idx) {
  Poly<K> P;
  const int n = FIXED ? K : poly_count(p.nv, idx, p.kmax);
  load_poly<K, FIXED>(p.xy, idx, p.kmax, p.vec4, n, P);
  Bounds b;
  b.x0 = b.x1 = P.x[0];
  b.y0 = b.y1 = P.y[0];
#pragma unroll
  for (int k = 1; k < K; ++k) {
    b.x0 = fminf(b.x0, P.x[k]);
    b.x1 = fmaxf(b.x1, P.x[k]);
    b.y0 = fminf(b.y0, P.y[k]);
    b.y1 = fmaxf(b.y1, P.y[k]);
  }
  b.lo = Z3 ? p.zlo[idx] : 0.f;
  b.hi = Z3 ? p.zhi[idx] : 0.f;
  return b;
}

__device__ __forceinline__ float lane_bcast(float v, int lane) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}

struct CullArgs {
  SegArgs seg;
  PolyArgs a, b;
  int64_t single_units;  // one block: its units
  int32_t* tile_count;
  int64_t tile_capacity;
  uint64_t* tile_mask;  // [tile_capacity][kMaskWords]
  int64_t* tile_prefix;   // [nseg+1] (segmented), written for the later kernels
  int64_t* group_prefix;  // [nseg+1]
  int* err;
};

constexpr int kBitWords = kTilePairs / 64;  // survivor bits of a tile
constexpr int kMaskWords = DGAL_TILE_MASK_WORDS;            // + tile origin + row length
static_assert(kMaskWords == kBitWords + 2 && kMaskWords <= 64, "mask words");

// Sign bit of the difference hi - lo: set when lo > hi, clear when they are
// equal (the closed test keeps touching boxes).
__device__ __forceinline__ uint32_t gap_bits(float hi, float lo) {
  return __float_as_uint(hi - lo);
}

// The largest float below v (finite v): lo < v <=> lo <= below(v), so the
// open z test becomes the closed one on a lowered upper end.
__device__ __forceinline__ float below(float v) {
  const uint32_t b = __float_as_uint(v);
  if ((b & 0x7fffffffu) == 0u) return -1.40129846e-45f;  // +-0 -> -denorm_min
  return __uint_as_float((int32_t)b > 0 ? b - 1u : b + 1u);
}

__device__ __forceinline__ int64_t wave_first(int64_t v) {
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)((uint64_t)v >> 32));
  return (int64_t)(((uint64_t)hi << 32) | lo);
}

// Quotient and remainder of a non-negative index by a positive divisor below
// 2^24 (32-bit division when the index allows it).
__device__ __forceinline__ void divmod(int64_t v, int64_t d, int64_t& q, int64_t& r) {
  if (v < (int64_t)0xffffffff) {
    const uint32_t q32 = (uint32_t)v / (uint32_t)d;
    q = q32;
  } else {
    q = v / d;
  }
  r = v - q * d;
}

// ---- the cull pass ----------------------------------------------------
// Survivor masks and counts, in units of 256 or 64 rows x one tile column of a
// segment.  The output's initial values are written by the list pass.
// 64 rows a wavefront, or (words) the same 64 rows for all of them
constexpr int unit_rows_of(bool words) { return words ? 64 : kCullBlock; }
constexpr int kBins = 32;              // bins per axis of the masks' broad phase
constexpr int kSparse = 16;            // most candidates of a word tested one by one
constexpr int kFillStep = 4 * kCullBlock;  // values a fill workgroup stores at once

// The pass's work in one segment (none where the segment is rejected).
__device__ __forceinline__ int64_t mask_units_of(const Segment& g, int rl, int unit_rows) {
  return (g.ok && g.na > 0 && g.nb > 0) ? (g.na + unit_rows - 1) / unit_rows * col_tiles_of(g, rl)
                                        : 0;
}
__device__ __forceinline__ int64_t fill_units_of(const Segment& g, const float* iou) {
  const int64_t mis = (int64_t)((reinterpret_cast<uintptr_t>(iou + g.out0) >> 2) & 3);
  return (g.ok && g.na > 0 && g.nb > 0) ? (g.na * g.nb + mis + kFillStep - 1) / kFillStep : 0;
}
__device__ __forceinline__ int64_t tiles_of(const Segment& g, int rl) {
  return g.ok ? tile_rows_of(g, rl) * col_tiles_of(g, rl) : 0;
}

// Exclusive prefixes over the segments of the workgroup's kind of units and
// of the tiles: thread t holds those at segment t * per.  Computed by every
// workgroup from the offsets (a few loads a thread), so that the pass needs
// no launch before it and no workspace.
struct SegScan {
  int64_t units[kCullBlock], tiles[kCullBlock];
  int64_t wave_sum[2][kCullBlock / 64];
  int64_t total;  // units of all segments
};

template <class F>
__device__ __forceinline__ void scan_segments(const SegArgs& a, SegScan& sc, F units_of) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int per = (a.nseg + kCullBlock - 1) / kCullBlock;
  const int s0 = min(a.nseg, tid * per), s1 = min(a.nseg, s0 + per);
  int64_t u = 0, t = 0;
  for (int s = s0; s < s1; ++s) {
    const Segment g = load_segment(a, s);
    u += units_of(g);
    t += tiles_of(g, a.rows_log2);
  }
  int64_t iu = u, it = t;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int64_t ou = __shfl_up(iu, d), ot = __shfl_up(it, d);
    if (lane >= d) {
      iu += ou;
      it += ot;
    }
  }
  if (lane == 63) {
    sc.wave_sum[0][wave] = iu;
    sc.wave_sum[1][wave] = it;
  }
  __syncthreads();
  for (int w = 0; w < wave; ++w) {
    iu += sc.wave_sum[0][w];
    it += sc.wave_sum[1][w];
  }
  sc.units[tid] = iu - u;
  sc.tiles[tid] = it - t;
  if (tid == kCullBlock - 1) sc.total = iu;
  __syncthreads();
}

// The workgroup's second scan: the segments' tile and row-group prefixes for
// the kernels that follow and for the backward; rejected segments own nothing
// and raise kErrSegment.  After the tile prefixes (when there is room) goes the
// size of the output, if the blocks cover it from 0 on without gaps, else -1.
__device__ __forceinline__ void write_prefixes(const CullArgs& m, SegScan& sc) {
  const SegArgs& a = m.seg;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int per = (a.nseg + kCullBlock - 1) / kCullBlock;
  const int s0 = min(a.nseg, tid * per), s1 = min(a.nseg, s0 + per);
  int64_t v = 0;
  bool dense = true;
  for (int s = s0; s < s1; ++s) {
    const Segment g = load_segment(a, s);
    if (g.ok) v += groups_of(g);
    else raise_error(m.err, kErrSegment);
    const int64_t next = s + 1 < a.nseg ? a.out_off[s + 1] : g.out0 + g.na * g.nb;
    dense = dense && g.ok && next == g.out0 + g.na * g.nb && (s > 0 || g.out0 == 0);
  }
  dense = __syncthreads_and(dense);
  if (s0 < s1 && s1 == a.nseg && a.nseg < kMaxSeg) {
    const Segment g = load_segment(a, a.nseg - 1);
    m.tile_prefix[a.nseg + 1] = dense ? g.out0 + g.na * g.nb : -1;
  }
  int64_t rg = v;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int64_t o = __shfl_up(rg, d);
    if (lane >= d) rg += o;
  }
  if (lane == 63) sc.wave_sum[0][wave] = rg;
  __syncthreads();
  for (int w = 0; w < wave; ++w) rg += sc.wave_sum[0][w];
  rg -= v;
  int64_t rt = sc.tiles[tid];
  if (tid == 0) {
    m.tile_prefix[0] = 0;
    m.group_prefix[0] = 0;
  }
  for (int s = s0; s < s1; ++s) {
    const Segment g = load_segment(a, s);
    if (g.ok) {
      rg += groups_of(g);
      rt += tiles_of(g, a.rows_log2);
    }
    m.tile_prefix[s + 1] = rt;
    m.group_prefix[s + 1] = rg;
  }
}

// Segment of unit u (u < total), its first unit and first tile.
struct UnitSeg {
  Segment g;
  int64_t unit0, tile0;
};

template <class F>
__device__ __forceinline__ UnitSeg find_unit(const SegArgs& a, const SegScan& sc, int64_t u,
                                             F units_of) {
  const int lane = threadIdx.x & 63;
  // the last thread whose prefix is not past u
  int k = -1;
#pragma unroll
  for (int q = 0; q < kCullBlock / 64; ++q)
    k += __popcll(__ballot(sc.units[q * 64 + lane] <= u));
  const int per = (a.nseg + kCullBlock - 1) / kCullBlock;
  UnitSeg r;
  r.unit0 = sc.units[k];
  r.tile0 = sc.tiles[k];
  const int s1 = min(a.nseg, k * per + per);
  for (int s = k * per;; ++s) {
    r.g = load_segment(a, s);
    const int64_t n = units_of(r.g);
    if (u < r.unit0 + n || s + 1 >= s1) break;
    r.unit0 += n;
    r.tile0 += tiles_of(r.g, a.rows_log2);
  }
  return r;
}

// Wave-wide minimum of v (every lane gets it), by data-parallel row moves.
__device__ __forceinline__ float wave_min(float v) {
#define DGAL_MIN_STEP(ctrl, rows)                                                            \
  v = fminf(v, __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(v), __float_as_int(v), \
                                                          ctrl, rows, 0xf, false)))
  DGAL_MIN_STEP(0x111, 0xf);  // row_shr:1, 2, 4, 8
  DGAL_MIN_STEP(0x112, 0xf);
  DGAL_MIN_STEP(0x114, 0xf);
  DGAL_MIN_STEP(0x118, 0xf);
  DGAL_MIN_STEP(0x142, 0xa);  // row_bcast:15 into rows 1 and 3
  DGAL_MIN_STEP(0x143, 0xc);  // row_bcast:31 into rows 2 and 3
#undef DGAL_MIN_STEP
  return lane_bcast(v, 63);
}

// Inclusive prefix OR over the lanes of each half of the wavefront.
__device__ __forceinline__ uint32_t half_prefix_or(uint32_t v) {
#define DGAL_OR_STEP(ctrl, rows) \
  v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, ctrl, rows, 0xf, false)
  DGAL_OR_STEP(0x111, 0xf);
  DGAL_OR_STEP(0x112, 0xf);
  DGAL_OR_STEP(0x114, 0xf);
  DGAL_OR_STEP(0x118, 0xf);
  DGAL_OR_STEP(0x142, 0xa);
#undef DGAL_OR_STEP
  return v;
}

// Bin of a coordinate: monotone in v for any lo and scale (a NaN product, an
// infinite scale times zero, counts as the lowest bin), so an order between
// coordinates is an order between their bins.
__device__ __forceinline__ int bin_of(float v, float lo, float scale) {
  return (int)fminf(fmaxf((v - lo) * scale, 0.f), (float)(kBins - 1));
}

template <bool Z3, int C, bool WORDS>
struct MaskLds {
  float4 xy[C];                         // the columns' bounds x0, y0, x1, y1
  float2 z[Z3 ? C : 1];                 // and z-extents, the upper end lowered
  // per axis and 64 columns: entry b < kBins holds the columns whose lower
  // end lies in bin b or below, entry kBins + b those whose upper end lies
  // in bin kBins - 1 - b or above
  uint64_t bm[Z3 ? 3 : 2][C / 64][2 * kBins];
  float2 bins[Z3 ? 3 : 2][C / 64];      // their first coordinate, and bins per unit length
  uint32_t count[WORDS ? kCullBlock / 64 : 1][64];  // the wavefronts' survivors of a row
};

// Masks of one unit: its rows from row r0 of segment g against the columns of
// tile column tc; a lane holds a row, and tests it against all words of 64
// columns, or (WORDS) its wavefront's share of them.  A pair survives when its
// closed boxes overlap (touching ones go to the exact kernel) and their open
// z extents do (the closed test on upper ends lowered by one ulp): the sign
// bits of its four (six) bound differences are all clear.  Only the pairs
// whose bins overlap on every axis are tested: the columns' bins are kept as
// bit sets, so that the two (three) axes cost a lane four (six) LDS reads for
// 64 columns, and on c5 leave about one pair of them to test.  A word's bins
// span the bounds of its own 64 columns: boxes laid out in an order have bins
// where they lie, and a far box costs one word its bins, not the tile.  A word
// that leaves a lane more than kSparse candidates (a far box, a crowd) is tested
// whole, every lane the same column, whose bounds are one LDS broadcast: no
// layout costs more than a test of every pair (a candidate alone takes some 200
// cycles of latency, two at a time; a column of all 7 to 10 vector
// instructions; kSparse 8 took 3% more on a 3D crowd, 24 the same).  Bound by
// latency (the LDS reads of the tests; the busiest lane has about four): 23 us
// on c5, 7 on 4096 x 4096.  Forwards of other layouts, in us: kernels that
// tested every pair and wrote the zeros / bins of the tile's first 64 columns
// for all of it / so:
//   4096 x 4096    random 39 / 30.5 / 30, sorted along x 38 / 34 / 30, in grid
//                  order 39 / 44 / 30, a far box every 256 39 / 35 / 31, every 64
//                  38 / 57 / 34, a crowd (10% overlap) 80 / 72 / 68
//   1000 x 1000    random 21 / 19.7 / 17, a crowd 23 / 27 / 20, a denser one (75%
//                  overlap) 42 / 72 / 41
//   64 3D scenes   random 156 / 114 / 114, sorted 149 / 116 / 113, far boxes
//                  160 / 128 / 118 and 157 / 185 / 140, a crowd 357 / 302 / 302
// Rows and columns past the block, and empty z extents, survive nothing.
template <int K, bool FIXED, bool Z3, int R, bool WORDS>
__device__ __forceinline__ void mask_unit(const CullArgs& m, const Segment& g, int64_t tile0,
                                          int64_t r0, int64_t tc,
                                          MaskLds<Z3, kTilePairs / R, WORDS>& s) {
  constexpr int C = kTilePairs / R, W = C / 64, D = Z3 ? 3 : 2, WAVES = kCullBlock / 64;
  constexpr int kUnroll = Z3 ? 4 : 8;
  constexpr int RL = R == 4 ? 2 : (R == 8 ? 3 : 4);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t cb = tc * C;
  const int nc = (int)min((int64_t)C, g.nb - cb);  // columns of the tile
  __syncthreads();  // the previous unit's reads are done
  for (int c = tid; c < C; c += kCullBlock) {
    Bounds b = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    if (c < nc) b = box_bounds<K, FIXED, Z3>(m.b, g.b0 + cb + c);
    if (Z3) {
      if (c >= nc || !(b.hi > b.lo)) {
        b.lo = __builtin_inff();  // marks a column that nothing meets
        b.hi = 0.f;
      }
      s.z[c] = make_float2(b.lo, below(b.hi));
    }
    s.xy[c] = make_float4(b.x0, b.y0, b.x1, b.y1);
  }
  for (int i = tid; i < D * W * 2 * kBins; i += kCullBlock) (&s.bm[0][0][0])[i] = 0ull;
  __syncthreads();
  for (int w = wave; w < W; w += WAVES) {  // each wavefront its own words
    const int c = w * 64 + lane;
    const float4 b = s.xy[c];
    float2 z = make_float2(0.f, 0.f);
    if constexpr (Z3) z = s.z[c];
    const bool in = c < nc && !(Z3 && z.x == __builtin_inff());
    const float l[3] = {b.x, b.y, z.x}, h[3] = {b.z, b.w, z.y};
    const uint64_t bit = 1ull << lane;
#pragma unroll
    for (int a = 0; a < D; ++a) {  // the bins span these 64 columns' bounds
      const float lo = wave_min(in ? l[a] : __builtin_inff());
      const float hi = -wave_min(in ? -h[a] : __builtin_inff());
      const float scale = (float)kBins * fast_rcp(hi - lo);
      if (lane == 0) s.bins[a][w] = make_float2(lo, scale);
      if (in) {
        __hip_atomic_fetch_or(&s.bm[a][w][bin_of(l[a], lo, scale)], bit, __ATOMIC_RELAXED,
                              __HIP_MEMORY_SCOPE_WORKGROUP);
        __hip_atomic_fetch_or(&s.bm[a][w][2 * kBins - 1 - bin_of(h[a], lo, scale)], bit,
                              __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      }
    }
    wave_sync();
#pragma unroll
    for (int a = 0; a < D; ++a) {
      const uint64_t v = s.bm[a][w][lane];
      s.bm[a][w][lane] = (uint64_t)half_prefix_or((uint32_t)(v >> 32)) << 32 |
                         half_prefix_or((uint32_t)v);
    }
  }
  __syncthreads();

  const int64_t row = r0 + (WORDS ? 0 : wave * 64) + lane;  // in the segment
  if (!WORDS && r0 + wave * 64 >= g.na) return;  // uniform in the wavefront
  Bounds rb = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if (row < g.na) rb = box_bounds<K, FIXED, Z3>(m.a, g.a0 + row);
  const bool live = row < g.na && !(Z3 && !(rb.hi > rb.lo));
  if (Z3) rb.hi = below(rb.hi);
  const float rl[3] = {rb.x0, rb.y0, rb.lo}, rh[3] = {rb.x1, rb.y1, rb.hi};
  const int64_t tr = row >> RL;
  const int64_t u = tile0 + tr * col_tiles_of(g, RL) + tc;
  const bool have = row < (tile_rows_of(g, RL) << RL) && u < m.tile_capacity;
  uint64_t* state = m.tile_mask + u * kMaskWords + (lane & (R - 1));
  uint32_t n = 0u;
#pragma unroll
  for (int i = 0; i < (WORDS ? (W + WAVES - 1) / WAVES : W); ++i) {
    const int w = WORDS ? wave + i * WAVES : i;
    if (WORDS && w >= W) break;  // uniform
    uint64_t keep = 0ull;
    if (w * 64 < nc) {  // uniform
      uint64_t cand = live ? ~0ull : 0ull;
      // columns that begin at or below the row's end, and end at or above its start
#pragma unroll
      for (int a = 0; a < D; ++a) {
        const float2 b = s.bins[a][w];
        cand &= s.bm[a][w][bin_of(rh[a], b.x, b.y)] &
                s.bm[a][w][2 * kBins - 1 - bin_of(rl[a], b.x, b.y)];
      }
      if (m.seg.self_pairs) {  // the diagonal
        const int64_t dd = row - (cb + w * 64);
        if (dd >= 0 && dd < 64) cand &= ~(1ull << dd);
      }
      // sign bit clear: column j and the row overlap
      auto gaps = [&](int j) {
        const float4 b = s.xy[j];
        uint32_t bits = gap_bits(rb.x1, b.x) | gap_bits(b.z, rb.x0) | gap_bits(rb.y1, b.y) |
                        gap_bits(b.w, rb.y0);
        if constexpr (Z3) {
          const float2 z = s.z[j];
          bits |= gap_bits(rb.hi, z.x) | gap_bits(z.y, rb.lo);
        }
        return bits;
      };
      if (__ballot(__popcll(cand) > kSparse) == 0ull) {  // uniform
        while (cand != 0ull) {  // the first and the last one left
          const int j = __builtin_ctzll(cand), k = 63 - __builtin_clzll(cand);
          const uint64_t bj = 1ull << j, bk = 1ull << k;
          const uint32_t gj = gaps(w * 64 + j), gk = gaps(w * 64 + k);
          if ((int32_t)gj >= 0) keep |= bj;
          if ((int32_t)gk >= 0) keep |= bk;
          cand &= ~(bj | bk);
        }
      } else {  // every column, the same in all lanes
        uint32_t half[2] = {0u, 0u};
#pragma unroll
        for (int h = 0; h < 2; ++h) {
#pragma unroll kUnroll
          for (int j = 31; j >= 0; --j)
            half[h] = __builtin_amdgcn_alignbit(half[h], gaps(w * 64 + h * 32 + j), 31);
        }
        keep = cand & ~((uint64_t)half[1] << 32 | half[0]);
      }
    }
    n += (uint32_t)__popcll(keep);
    if (have) state[w * R] = keep;
  }
  if constexpr (WORDS) {
    s.count[wave][lane] = n;
    __syncthreads();
    if (wave != 0) return;
    n = 0u;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) n += s.count[w][lane];
  }
  // the tile's count: its R rows are R neighbouring lanes
#pragma unroll
  for (int d = 1; d < R; d <<= 1) n += (uint32_t)__shfl_xor((int)n, d);
  if ((lane & (R - 1)) == 0 && row < g.na) {
    if (have) {
      m.tile_count[u] = (int32_t)n;
      state[kBitWords] = (uint64_t)(g.out0 + row * g.nb + cb);
      state[kBitWords + 1] = (uint64_t)g.nb;
    } else {
      raise_error(m.err, kErrCapacity);
    }
  }
}

template <int K, bool FIXED, bool Z3, int R, bool WORDS>
__global__ __launch_bounds__(kCullBlock)
__attribute__((amdgpu_waves_per_eu(R == 4 || !Z3 ? 5 : 7))) void k_matrix_cull(CullArgs m) {
  static_assert(R == 4 || R == 8 || R == 16, "tile rows");
  constexpr int C = kTilePairs / R;
  constexpr int RL = R == 4 ? 2 : (R == 8 ? 3 : 4);
  constexpr int UNIT_ROWS = unit_rows_of(WORDS);
  __shared__ MaskLds<Z3, C, WORDS> s_mask;
  __shared__ SegScan s_scan;
  const bool segmented = m.seg.a_off != nullptr;
  auto units_of = [&](const Segment& g) { return mask_units_of(g, RL, UNIT_ROWS); };
  UnitSeg us = {load_segment(m.seg, 0), 0, 0};
  int64_t total = m.single_units;
  if (segmented) {
    scan_segments(m.seg, s_scan, units_of);
    total = s_scan.total;
    if (blockIdx.x == 0) write_prefixes(m, s_scan);
  }
  for (int64_t u = blockIdx.x; u < total; u += gridDim.x) {
    if (segmented) us = find_unit(m.seg, s_scan, u, units_of);
    const int64_t nct = col_tiles_of(us.g, RL);
    int64_t rc, tc;
    divmod(u - us.unit0, nct, rc, tc);
    mask_unit<K, FIXED, Z3, R, WORDS>(m, us.g, us.tile0, rc * UNIT_ROWS, tc, s_mask);
  }
}

// Sums of the tile counts over chunks of kScanChunk tiles, for tables too large
// for every workgroup of the list pass to sum the counts before its own.
constexpr int kScanChunk = kScanBlock * 4;

__device__ __forceinline__ int64_t scan_tiles(const int64_t* tile_prefix, int nseg,
                                              int64_t single_tiles, int64_t tile_capacity) {
  const int64_t nt = tile_prefix != nullptr ? tile_prefix[nseg] : single_tiles;
  return nt < tile_capacity ? nt : tile_capacity;
}

// Block-wide inclusive scan of one value per thread (wave scans + LDS).
__device__ __forceinline__ int64_t block_inclusive_scan(int64_t v, int64_t* s_w) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int64_t o = __shfl_up(v, d);
    if (lane >= d) v += o;
  }
  if (lane == 63) s_w[wave] = v;
  __syncthreads();
  int64_t add = 0;
  for (int w = 0; w < wave; ++w) add += s_w[w];
  __syncthreads();
  return v + add;
}

__global__ __launch_bounds__(kScanBlock) void k_scan_totals(const int64_t* tile_prefix, int nseg,
                                                            int64_t single_tiles,
                                                            int64_t tile_capacity,
                                                            const int32_t* tile_count,
                                                            int64_t* totals) {
  __shared__ int64_t s_w[kScanBlock / 64];
  const int64_t nt = scan_tiles(tile_prefix, nseg, single_tiles, tile_capacity);
  const int64_t c0 = (int64_t)blockIdx.x * kScanChunk;
  if (c0 >= nt) return;  // uniform
  int64_t v = 0;
#pragma unroll
  for (int k = 0; k < kScanChunk / kScanBlock; ++k) {
    const int64_t t = c0 + k * kScanBlock + threadIdx.x;
    if (t < nt) v += tile_count[t];
  }
  v = block_inclusive_scan(v, s_w);
  if (threadIdx.x == kScanBlock - 1) totals[blockIdx.x] = v;
}

struct ListArgs {
  SegArgs seg;
  int64_t single_tiles;
  float* iou;
  int64_t list_blocks;  // workgroups of the list; the others fill the output
  int64_t tile_capacity;
  const int32_t* tile_count;
  const int64_t* totals;  // sums of the chunks of kScanChunk tiles, or NULL
  const uint64_t* tile_mask;
  int64_t* tile_start;
  int64_t* pair_id;
  int64_t capacity;
  int64_t* count;
  int* err;
};

// ---- the work list ------------------------------------------------------
// Sum of the counts of tiles [0, t) by a workgroup of kListBlock threads
// (every thread gets it): whole chunks from the totals when they were taken
// (large tables), the rest from the counts, 16 bytes a load when aligned.
__device__ __forceinline__ int64_t sum_before(const int32_t* cnt, const int64_t* totals, int64_t t,
                                              int64_t* s_w) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int64_t first = 0, v = 0;
  if (totals != nullptr) {
    const int64_t chunks = t / kScanChunk;
    for (int64_t k = tid; k < chunks; k += kListBlock) v += totals[k];
    first = chunks * kScanChunk;
  }
  if ((reinterpret_cast<uintptr_t>(cnt) & 15) == 0) {  // uniform (chunks are multiples of 4)
    const int64_t n4 = (t - first) >> 2;
    const int4* c4 = reinterpret_cast<const int4*>(cnt + first);
    int64_t k = tid;
    for (; k + 3 * kListBlock < n4; k += 4 * kListBlock) {  // four loads in flight
      const int4 a = c4[k], b = c4[k + kListBlock], c = c4[k + 2 * kListBlock],
                 d = c4[k + 3 * kListBlock];
      v += (int64_t)(a.x + a.y + a.z + a.w) + (b.x + b.y + b.z + b.w) + (c.x + c.y + c.z + c.w) +
           (d.x + d.y + d.z + d.w);
    }
    for (; k < n4; k += kListBlock) {
      const int4 a = c4[k];
      v += a.x + a.y + a.z + a.w;
    }
    first += n4 << 2;
  }
  for (int64_t k = first + tid; k < t; k += kListBlock) v += cnt[k];
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) v += __shfl_xor(v, d);
  if (lane == 0) s_w[wave] = v;
  __syncthreads();
  v = 0;
#pragma unroll
  for (int w = 0; w < kListBlock / 64; ++w) v += s_w[w];
  __syncthreads();
  return v;
}

// A wavefront's step of the fill: zeros to values [o, o + 256) of the `size`
// ones at out (o may be below 0, and the last step past the end), four a lane,
// o chosen so that each lane's four are one aligned store.
__device__ __forceinline__ void fill_step(float* out, int64_t size, int64_t o) {
  const int64_t e = o + 4 * (threadIdx.x & 63);
  if (e >= 0 && e + 4 <= size) {
    *reinterpret_cast<float4*>(out + e) = make_float4(0.f, 0.f, 0.f, 0.f);
  } else {  // the first or last values
#pragma unroll
    for (int c = 0; c < 4; ++c)
      if (e + c >= 0 && e + c < size) out[e + c] = 0.f;
  }
}

// The output's zeros (the exact kernel, later, writes the survivors and the
// self diagonals over them), by the list pass's other workgroups: the list is
// bound by latency and the fill by memory, so they share the chip.  Where the
// blocks cover the output without gaps it is one flat stream, a step a
// workgroup: one aligned 16-byte store a lane and short-lived wavefronts
// write 6.7 TB/s here (348 MB alone in 52 us, c5's 374 MB beside the list in
// 62; grid-stride loops 5.6, and the rows of the masks' tiles, as the masks were
// made, 3.9, each row ending in two partial cache lines).  Otherwise each block is filled by itself, found from
// a scan of the segments, and gaps are left alone.
__device__ __forceinline__ void fill_output(const ListArgs& m, int64_t b, int64_t nblk,
                                            SegScan& sc) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const SegArgs& a = m.seg;
  int64_t size = a.a_count * a.b_count;
  if (a.a_off != nullptr) size = a.nseg < kMaxSeg ? m.seg.tile_prefix[a.nseg + 1] : -1;
  if (size >= 0) {
    const int mis = (int)((reinterpret_cast<uintptr_t>(m.iou) >> 2) & 3);
    for (int64_t o = b * kFillStep + wave * 256 - mis; o < size; o += nblk * kFillStep)
      fill_step(m.iou, size, o);
    return;
  }
  nblk = min(nblk, (int64_t)kFillSegBlocks);
  if (b >= nblk) return;  // uniform
  auto units_of = [&](const Segment& g) { return fill_units_of(g, m.iou); };
  scan_segments(a, sc, units_of);
  for (int64_t u = b; u < sc.total; u += nblk) {
    const UnitSeg us = find_unit(a, sc, u, units_of);
    float* out = m.iou + us.g.out0;
    const int mis = (int)((reinterpret_cast<uintptr_t>(out) >> 2) & 3);
    fill_step(out, us.g.na * us.g.nb, (u - us.unit0) * kFillStep + wave * 256 - mis);
  }
}

// Lays out the work list: the exclusive prefix of the tile counts, and the
// survivors' output indices from the tile state the cull wrote (bits,
// origin, row length), each tile's in the order of its bits (chunk-major).  A
// workgroup takes a contiguous range of tiles, whose start it sums from the
// counts before it, and walks it kListTiles tiles at a time: a scan of their
// counts, then two tiles a wavefront step, a lane for each word of bits.
// One launch in place of two or three (the scan's and this one's own): bound
// by latency, and the sums are L2 reads (c5: 45.7 k counts, 183 KB).
__global__ __launch_bounds__(kListBlock) void k_matrix_list(ListArgs m) {
  __shared__ SegScan s_scan;
  constexpr int WAVES = kListBlock / 64;
  __shared__ int64_t s_w[WAVES];
  __shared__ int64_t s_start[kListTiles];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  if ((int64_t)blockIdx.x >= m.list_blocks) {
    fill_output(m, (int64_t)blockIdx.x - m.list_blocks, (int64_t)gridDim.x - m.list_blocks, s_scan);
    return;
  }
  int64_t nt = m.seg.a_off != nullptr ? m.seg.tile_prefix[m.seg.nseg] : m.single_tiles;
  nt = nt < m.tile_capacity ? nt : m.tile_capacity;
  const int64_t per = (nt + m.list_blocks - 1) / m.list_blocks;
  const int64_t t0 = blockIdx.x * per, t1 = min(nt, t0 + per);
  if (t0 >= t1) {  // uniform; an empty matrix still publishes its total
    if (blockIdx.x == 0 && tid == 0) *m.count = 0;
    return;
  }
  int64_t run = sum_before(m.tile_count, m.totals, t0, s_w);
  for (int64_t b0 = t0; b0 < t1; b0 += kListTiles) {
    const int nb_tiles = (int)min((int64_t)kListTiles, t1 - b0);
    // one tile a thread: wave scan, then the waves before it
    const int c = tid < nb_tiles ? m.tile_count[b0 + tid] : 0;
    int incl = c;  // at most kListTiles * 2048
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const int o = __shfl_up(incl, d);
      if (lane >= d) incl += o;
    }
    if (lane == 63) s_w[wave] = incl;
    __syncthreads();
    int64_t start = run + incl - c;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
      if (w < wave) start += s_w[w];
      run += s_w[w];
    }
    s_start[tid] = start;
    if (tid < nb_tiles) m.tile_start[b0 + tid] = start;
    __syncthreads();
    const int word = lane & (kBitWords - 1);
    const int rl = m.seg.rows_log2;
    const int j = word & ((1 << rl) - 1), ch = word >> rl;
    uint64_t bits_next = 0ull;
    int64_t origin_next = 0, nb_next = 0;
    auto load = [&](int k) {
      const bool in = k + (lane >> 5) < nb_tiles;
      const uint64_t* st = m.tile_mask + (b0 + k + (lane >> 5)) * kMaskWords;
      bits_next = in ? st[word] : 0ull;
      origin_next = in ? (int64_t)st[kBitWords] : 0;
      nb_next = in ? (int64_t)st[kBitWords + 1] : 0;
    };
    load(wave * 2);
    for (int k = wave * 2; k < nb_tiles; k += 2 * WAVES) {  // uniform
      const uint64_t bits = bits_next;
      const int64_t first = origin_next + (int64_t)j * nb_next + ch * 64;
      load(k + 2 * WAVES);  // the next two tiles' state
      // the word's first slot: the exclusive prefix of the words' bit counts
      const int cnt = __popcll(bits);
      int pre = cnt;
#pragma unroll
      for (int d = 1; d < kBitWords; d <<= 1) {
        const int o = __shfl_up(pre, d, kBitWords);
        if (word >= d) pre += o;
      }
      int64_t slot = s_start[min(k + (lane >> 5), kListTiles - 1)] + (pre - cnt);
      uint64_t w = bits;
      while (w != 0ull) {
        const int b = __builtin_ctzll(w);
        w &= w - 1ull;
        if (slot < m.capacity) m.pair_id[slot] = first + b;
        ++slot;
      }
    }
    __syncthreads();  // s_start is the next round's
  }
  if (t1 == nt && tid == 0) {
    *m.count = run;
    if (run > m.capacity) raise_error(m.err, kErrCapacity);
  }
}
struct ExactArgs {
  SegArgs seg;
  PolyArgs a, b;
  float* iou;
  const int64_t* pair_id;
  uint8_t* s_nx;
  uint8_t* s_flags;
  int64_t capacity;
  const int64_t* count;
  int cap;
  bool flags_vec;  // cap == 2K and s_flags aligned to cap bytes: whole-row stores
  int* err;
  unsigned long long* stats;  // path statistics (NULL: off)
  // an overflowing list's tile counts are cut to its capacity here
  const int64_t* tile_start;
  int32_t* tile_count;
  int64_t tile_capacity;
  int64_t single_tiles;
};

// Segment, row and column (within the segment) of a flat output index.  The
// work list is in output order, so the entries of one wavefront mostly share
// a segment: it is searched once for the wavefront's first entry, and a lane
// outside that segment searches for itself.
// The segment a wavefront last located, and its block of the output
// [lo, hi) (empty until the first search; wave-uniform).
struct SegCache {
  Segment g;
  int64_t lo = 0, hi = 0;
};

__device__ __forceinline__ bool locate(const SegArgs& sa, int64_t pid, SegCache& sc, Segment& g,
                                       int64_t& r, int64_t& c) {
  if (sa.a_off == nullptr) {
    g = load_segment(sa, 0);
  } else {
    const int64_t pid0 = wave_first(pid);
    if (!(pid0 >= sc.lo && pid0 < sc.hi)) {  // uniform: a wavefront's entries mostly stay in one
      sc.g = load_segment(sa, wave_find_segment(sa.out_off, sa.nseg, pid0));
      sc.lo = sc.g.out0;
      sc.hi = sc.g.ok ? sc.g.out0 + sc.g.na * sc.g.nb : sc.g.out0;
    }
    g = (pid >= sc.lo && pid < sc.hi) ? sc.g : load_segment(sa, find_segment(sa.out_off, sa.nseg, pid));
  }
  const int64_t local = pid - g.out0;
  if (!g.ok || g.nb <= 0 || local < 0) return false;
  divmod(local, g.nb, r, c);
  return r < g.na;
}

// The 1s on the diagonals of self blocks, a row a thread, by the last
// workgroups of the exact pass (the ones that most often have no entries).  The
// rows are found by their row groups, which only the accepted segments own: a
// rejected one's offsets need not be in order, so a row's place in a_off does
// not tell its segment.
__device__ __forceinline__ void write_diagonals(const SegArgs& a, int64_t groups, float* iou) {
  const bool segmented = a.a_off != nullptr;
  const int64_t threads = (int64_t)gridDim.x * kExactBlock;
  for (int64_t t0 = ((int64_t)gridDim.x - 1 - blockIdx.x) * kExactBlock + (threadIdx.x & ~63);
       t0 < groups * kGroupRows; t0 += threads) {  // the wavefront's 64 rows
    const int64_t u = (t0 + (threadIdx.x & 63)) / kGroupRows;
    const int s0 =
        segmented ? wave_find_segment(a.group_prefix, a.nseg, wave_first(t0 / kGroupRows)) : 0;
    if (u >= groups) continue;
    Segment g = load_segment(a, s0);
    int64_t first = 0;
    if (segmented) {
      first = a.group_prefix[s0];
      if (u >= a.group_prefix[s0 + 1]) {
        const int s = find_segment(a.group_prefix, a.nseg, u);
        g = load_segment(a, s);
        first = a.group_prefix[s];
      }
    }
    const int64_t r = (u - first) * kGroupRows + (threadIdx.x & (kGroupRows - 1));
    if (g.ok && r < g.na) iou[g.out0 + r * (g.nb + 1)] = 1.f;
  }
}

template <int K, bool FIXED, bool Z3>
__global__ __launch_bounds__(kExactBlock)
__attribute__((amdgpu_waves_per_eu(4))) void k_matrix_exact(ExactArgs m) {
  constexpr int CAP = 2 * K;
  __shared__ float2 s_pt[CAP * kExactBlock];
  __shared__ uint16_t s_cd[CAP * kExactBlock];
  const int tid = threadIdx.x;
  int64_t n = *m.count;
  int64_t groups = 0;  // row groups with a diagonal
  if (m.seg.self_pairs)
    groups = m.seg.a_off != nullptr ? m.seg.group_prefix[m.seg.nseg]
                                    : (m.seg.a_count + kGroupRows - 1) / kGroupRows;
  if (n > m.capacity) {  // uniform; an overflow
    n = m.capacity;
    int64_t nt = m.seg.tile_prefix != nullptr ? m.seg.tile_prefix[m.seg.nseg] : m.single_tiles;
    nt = nt < m.tile_capacity ? nt : m.tile_capacity;
    for (int64_t t = (int64_t)blockIdx.x * kExactBlock + tid; t < nt;
         t += (int64_t)gridDim.x * kExactBlock) {
      const int64_t room = max((int64_t)0, m.capacity - m.tile_start[t]);
      if (room < m.tile_count[t]) m.tile_count[t] = (int32_t)room;
    }
  }
  if (groups > 0) write_diagonals(m.seg, groups, m.iou);
  // each wavefront a contiguous range of entries, 64 at a time: consecutive
  // entries mostly share a segment, which is then searched once
  const int64_t wid = ((int64_t)blockIdx.x * kExactBlock + tid) >> 6;
  const int64_t nw = ((int64_t)gridDim.x * kExactBlock) >> 6;
  const int64_t per = (((n + nw - 1) / nw) + 63) & ~(int64_t)63;
  const int64_t e_end = min(n, wid * per + per);
  SegCache sc;
  // 4-slot pairs: the next step's ids are loaded while this step's pairs are
  // evaluated (the 8-slot kernel has no registers to spare for them)
  constexpr bool PREFETCH = K == 4;
  int64_t pid_next = 0;
  if (PREFETCH && wid * per + (tid & 63) < e_end) pid_next = m.pair_id[wid * per + (tid & 63)];
  // (at K = 8 wavefronts stay whole for the pair forward: lanes without an
  // entry repeat the wavefront's last one, and their results are dropped)
  for (int64_t e = wid * per + (tid & 63); K == 8 ? e - (tid & 63) < e_end : e < e_end; e += 64) {
    bool live = K != 8 || e < e_end;
    const int64_t pid = PREFETCH ? pid_next : m.pair_id[live ? e : e_end - 1];
    if (PREFETCH && e + 64 < e_end) pid_next = m.pair_id[e + 64];
    Segment g;
    int64_t r = 0, c = 0;
    if (!locate(m.seg, pid, sc, g, r, c)) {  // not written by the cull on these shapes
      if (K != 8) continue;
      live = false;
      g.a0 = g.b0 = r = c = 0;
    }
    int64_t ia = g.a0 + r, ib = g.b0 + c;
    if (m.seg.self_pairs && r > c) {  // one unordered pair: the lower index is P
      const int64_t t = ia;
      ia = ib;
      ib = t;
    }
    const int n1 = FIXED ? K : poly_count(m.a.nv, ia, m.a.kmax);
    const int n2 = FIXED ? K : poly_count(m.b.nv, ib, m.b.kmax);
    Poly<K> P, Q;
    load_poly<K, FIXED>(m.a.xy, ia, m.a.kmax, m.a.vec4, n1, P);
    load_poly<K, FIXED>(m.b.xy, ib, m.b.kmax, m.b.vec4, n2, Q);
    PairResult<K> res;
    pair_forward<K, FIXED, kExactBlock>(P, n1, Q, n2, s_pt + tid, s_cd + tid, res, nullptr, live);
    if (!live) continue;
    count_path(m.stats, res.exact, res.thin);
    // (the list pass wrote the zeros; a third of c5's entries are disjoint, and
    // a scattered store costs its whole cache line)
    const float v = pair_iou<Z3>(res.inter, res.a1, res.a2, res.m, m.a.zlo, m.a.zhi, ia, m.b.zlo,
                                 m.b.zhi, ib);
    if (__float_as_uint(v) != 0u) m.iou[pid] = v;
    if (res.overflow) raise_error(m.err, kErrCapacity);
    m.s_nx[e] = (uint8_t)res.m;
    uint8_t* row = m.s_flags + e * (int64_t)m.cap;
    if (m.flags_vec) {  // uniform: a whole row in one store
      if constexpr (K == 4) {
        *reinterpret_cast<uint2*>(row) = make_uint2(res.codes[0], res.codes[1]);
      } else {
        *reinterpret_cast<uint4*>(row) =
            make_uint4(res.codes[0], res.codes[1], res.codes[2], res.codes[3]);
      }
    } else {
#pragma unroll
      for (int b = 0; b < CAP; ++b)
        if (b < m.cap) row[b] = (uint8_t)(res.codes[b >> 2] >> ((b & 3) * 8));
    }
    // rare: the areas again in fp64, from the polygons reloaded, and the IoU
    // written again
    if (res.thin) {
      load_poly<K, FIXED>(m.a.xy, opaque(ia), m.a.kmax, m.a.vec4, n1, P);
      load_poly<K, FIXED>(m.b.xy, opaque(ib), m.b.kmax, m.b.vec4, n2, Q);
      stage_pair<K, kExactBlock>(s_pt + tid, P, Q);
      float inter, a1, a2;
      thin_areas64<K, FIXED, kExactBlock>(res.m, res.codes, n1, n2, s_pt + tid, inter, a1, a2);
      m.iou[pid] = pair_iou<Z3>(inter, a1, a2, res.m, m.a.zlo, m.a.zhi, ia, m.b.zlo, m.b.zhi, ib);
    }
  }
}

// Zero-fills n floats.
__global__ void k_fill_zero(float* p, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    p[i] = 0.f;
}

struct BwdArgs {
  SegArgs seg;
  PolyArgs a, b;
  int64_t single_groups;
  const float* grad;
  const int64_t* pair_id;
  const uint8_t* s_nx;
  const uint8_t* s_flags;
  int64_t capacity;
  const int64_t* tile_start;
  const int32_t* tile_count;
  int64_t tile_capacity;
  int cap;
  bool flags_vec;  // cap == 2K and s_flags aligned to cap bytes: whole-row loads
  float* ga_xy;
  float* gb_xy;  // unused when self_pairs
  float* ga_z;
  float* gb_z;
};

template <int K>
constexpr int bwd_block() {
  return K == 8 ? 128 : 256;
}

// Sums one step's row gradients (64 entries, each one row's H value pairs:
// a vertex's x and y, or the z-extent's two ends) per (row, pair) into the
// lanes' accumulators without atomics (LDS float atomic adds measured slow
// here: 10 a lane per step cost the c5 backward ~15 us).  The lanes' pairs go
// to the wavefront's own LDS columns ordered by row (the row's offset, then
// the lane's rank among that row's lanes); lane c then adds up the run of
// combination c = (row c / H, pair c % H), and c + 64, ..., in lane order: a
// fixed order, so the sums are the same from run to run.  rl < 0: the lane
// holds nothing.  Called by all 64 lanes.
template <int H, int BLOCK>
__device__ __forceinline__ void step_row_sums(int rl, const float2 (&gv)[H], float2* stage,
                                              float2 (&acc)[(kGroupRows * H + 63) / 64]) {
  constexpr int NACC = (kGroupRows * H + 63) / 64;
  const int lane = threadIdx.x & 63;
  int pos = 0, base = 0, most = 0;
  int off[kGroupRows], cnt[kGroupRows];
#pragma unroll
  for (int r = 0; r < kGroupRows; ++r) {
    const uint64_t mr = __ballot(rl == r);
    const int c = __popcll(mr);
    if (rl == r)
      pos = base + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mr >> 32),
                                                  __builtin_amdgcn_mbcnt_lo((uint32_t)mr, 0u));
    off[r] = base;
    cnt[r] = c;
    base += c;
    most = max(most, c);
  }
  if (base == 0) return;  // uniform: nothing in this step
  if (rl >= 0) {
#pragma unroll
    for (int h = 0; h < H; ++h) stage[h * BLOCK + pos] = gv[h];
  }
  wave_sync();
#pragma unroll
  for (int j = 0; j < NACC; ++j) {
    const int c = lane + 64 * j;
    const int r = c / H, h = c - r * H;
    int o = 0, n = 0;  // the run of row r (none past the last row)
#pragma unroll
    for (int rr = 0; rr < kGroupRows; ++rr) {
      if (r == rr) {
        o = off[rr];
        n = cnt[rr];
      }
    }
    const float2* run = stage + h * BLOCK + o;
    float sx = 0.f, sy = 0.f;
    for (int i = 0; i < most; ++i) {
      if (i < n) {
        const float2 v = run[i];
        sx += v.x;
        sy += v.y;
      }
    }
    acc[j].x += sx;
    acc[j].y += sy;
  }
  wave_sync();  // the columns are the pair kernels' staging again
}

// One step's column gradients wait in the LDS columns of their lanes: K
// vertices, the z-extent's ends, the row of the second set and its vertex count.
template <int K, int BLOCK>
__device__ __forceinline__ void stage_column(float2* col, const float2 (&gq)[K], float2 gz,
                                             int64_t row, int n) {
#pragma unroll
  for (int k = 0; k < K; ++k) col[k * BLOCK] = gq[k];
  col[K * BLOCK] = gz;
  col[(K + 1) * BLOCK] = make_float2(__int_as_float((int)row), __int_as_float((int)(row >> 32)));
  col[(K + 2) * BLOCK].x = __int_as_float(n);
}

// Adds them to the second set's gradients; `live`: the lanes that staged one.
// A row's floats go to consecutive lanes, so that an instruction's atomic adds
// meet 8 (K = 8: 4) rows' cache lines and not 64: the adds leave the XCD, and
// the lines bound the kernel where a lane added its own row's floats one by one
// (4096 x 4096: 70 us, 38 so).  Called by all 64 lanes.
template <int K, bool FIXED, bool Z3, int BLOCK>
__device__ __forceinline__ void add_columns(uint64_t live, const float2* stage, float* gb_xy,
                                            int kmax, float* gb_z) {
  constexpr int L = 2 * K, E = 64 / L;  // floats of a row, rows an instruction takes
  static_assert(K + 3 <= 2 * K, "a staged column fits");
  if (live == 0) return;  // uniform
  const int lane = (int)opaque((int64_t)(threadIdx.x & 63));  // nothing of it kept between steps
  const float* flat = reinterpret_cast<const float*>(stage);
  auto row_of = [&](int e) {
    const float2 r = stage[(K + 1) * BLOCK + e];
    return (int64_t)(((uint64_t)(uint32_t)__float_as_int(r.y) << 32) |
                     (uint32_t)__float_as_int(r.x));
  };
  wave_sync();
  for (int j = 0; j < L; ++j) {
    const int e = j * E + lane / L, c = lane % L;
    if ((live >> e) & 1u) {
      const int n = FIXED ? K : __float_as_int(stage[(K + 2) * BLOCK + e].x);
      if (c < 2 * n)
        unsafeAtomicAdd(gb_xy + row_of(e) * (2 * kmax) + c,
                        flat[((c >> 1) * BLOCK + e) * 2 + (c & 1)]);
    }
  }
  if (Z3) {
    for (int j = 0; j < 2; ++j) {
      const int e = j * 32 + lane / 2, c = lane & 1;
      if ((live >> e) & 1u)
        unsafeAtomicAdd(gb_z + row_of(e) * 2 + c, flat[(K * BLOCK + e) * 2 + c]);
    }
  }
  wave_sync();  // the columns are the pair kernels' staging again
}

// SELF: self pairs; SPLIT: a workgroup for each row group (matrix_bwd_split).
// Kernels of their own: the roles' code together spilled, and the split as a
// run-time switch took the others 1 to 4% (32 scenes of 2D quadrilaterals 14.5
// us, 14.1 so; c5 44.9 and 44.5 in a graph).
template <int K, bool FIXED, bool Z3, bool SELF, bool SPLIT>
__global__ __launch_bounds__(bwd_block<K>())
__attribute__((amdgpu_waves_per_eu(K == 4 ? 4 : 2))) void k_matrix_bwd(BwdArgs m) {
  constexpr int BLOCK = bwd_block<K>();
  constexpr int WAVES = BLOCK / 64;
  constexpr int CAP = 2 * K;
  constexpr int H = K + (Z3 ? 1 : 0);  // a row's value pairs: vertices, then (zlo, zhi)
  constexpr int NACC = (kGroupRows * H + 63) / 64;
  static_assert(H <= CAP, "a step's row values fit the staging columns");
  __shared__ float2 s_v[CAP * BLOCK];
  __shared__ float2 s_g[CAP * BLOCK];
  __shared__ uint2 s_tab[256];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // uniform: the row-group walk is scalar
  float2* stage = s_v + wave * 64;  // this wavefront's columns of the staging
  fill_code_table<K, FIXED, BLOCK>(s_tab);
  __syncthreads();
  const bool segmented = m.seg.a_off != nullptr;
  const int64_t total = segmented ? m.seg.group_prefix[m.seg.nseg] : m.single_groups;
  const int kx = m.a.kmax;
  if (segmented) {
    // rows that no row group writes are zeroed here: rows outside every
    // segment, and the rows of a segment without row groups (rejected, or
    // without columns); every other row is written once by its row group
    const int64_t rowlen = (int64_t)kx * 2;
    auto zero_rows = [&](int64_t r0, int64_t r1, int64_t t, int64_t nt) {
      r0 = max(r0, (int64_t)0);
      r1 = min(r1, m.a.count);
      for (int64_t i = r0 * rowlen + t; i < r1 * rowlen; i += nt) m.ga_xy[i] = 0.f;
      if (Z3)
        for (int64_t i = r0 * 2 + t; i < r1 * 2; i += nt) m.ga_z[i] = 0.f;
    };
    const int64_t gt = (int64_t)blockIdx.x * BLOCK + tid, gn = (int64_t)gridDim.x * BLOCK;
    zero_rows(0, m.seg.a_off[0], gt, gn);
    zero_rows(m.seg.a_off[m.seg.nseg], m.a.count, gt, gn);
    for (int s = blockIdx.x; s < m.seg.nseg; s += gridDim.x)
      if (m.seg.group_prefix[s + 1] == m.seg.group_prefix[s])
        zero_rows(m.seg.a_off[s], m.seg.a_off[s + 1], tid, BLOCK);
  }

  // split: the workgroup's wavefronts take the group's steps in turn
  const int part = SPLIT ? wave : 0, parts = SPLIT ? WAVES : 1;
  const int64_t u0 = SPLIT ? blockIdx.x : (int64_t)blockIdx.x * WAVES + wave;
  for (int64_t u = u0; u < total; u += (int64_t)gridDim.x * WAVES) {
    const int s = segmented ? wave_find_segment(m.seg.group_prefix, m.seg.nseg, u) : 0;
    const int64_t tr = segmented ? u - m.seg.group_prefix[s] : u;  // row group in the segment
    const Segment g = load_segment(m.seg, s);
    if (!g.ok) continue;
    const int64_t r0 = tr * kGroupRows;
    const int nr = (int)min((int64_t)kGroupRows, g.na - r0);
    // the tile rows that cover the group (several when tiles are shorter
    // than the group, part of one when taller: entries of its other rows are
    // skipped below); their tiles are consecutive, so are their entries
    const int rlog = m.seg.rows_log2;
    const int64_t nct = col_tiles_of(g, rlog);
    const int64_t tbase = segmented ? m.seg.tile_prefix[s] : 0;
    const int64_t t0 = tbase + (r0 >> rlog) * nct;
    const int64_t t1 = tbase + (((r0 + nr - 1) >> rlog) + 1) * nct - 1;
    const bool have = t1 < m.tile_capacity;
    const int64_t e_begin = have ? m.tile_start[t0] : 0;
    const int64_t e_end = have ? m.tile_start[t1] + m.tile_count[t1] : 0;
    float2 acc[NACC];
#pragma unroll
    for (int j = 0; j < NACC; ++j) acc[j] = make_float2(0.f, 0.f);
    // one entry: its row in the group and the row box's gradient in gv
    // (every slot written), or -1 (gv untouched); of two sets also
    // stages the column box's
    auto entry = [&](int64_t e, float2 (&gv)[H]) -> int {
      if (e < 0 || e >= e_end || e >= m.capacity) return -1;
      // the entry's saved state in one round of loads (none waits for another)
      const int nx = m.s_nx[e];
      const int64_t pid = m.pair_id[e];
      const uint8_t* row = m.s_flags + e * (int64_t)m.cap;
      uint32_t codes[K / 2];
      if (m.flags_vec) {
        if constexpr (K == 4) {
          const uint2 w = *reinterpret_cast<const uint2*>(row);
          codes[0] = w.x;
          codes[1] = w.y;
        } else {
          const uint4 w = *reinterpret_cast<const uint4*>(row);
          codes[0] = w.x;
          codes[1] = w.y;
          codes[2] = w.z;
          codes[3] = w.w;
        }
      } else {
#pragma unroll
        for (int w = 0; w < K / 2; ++w) codes[w] = 0xffffffffu;
#pragma unroll
        for (int k = 0; k < CAP; ++k) {
          if (k < m.cap) {
            const uint32_t cc = row[k];
            codes[k >> 2] = (codes[k >> 2] & ~(0xffu << ((k & 3) * 8))) | (cc << ((k & 3) * 8));
          }
        }
      }
      if (nx == 0) return -1;  // empty intersection: zero gradient
      const int64_t local = pid - g.out0;
      if (local < 0 || g.nb <= 0) return -1;
      int64_t rg, col;  // row and column within the segment
      divmod(local, g.nb, rg, col);
      const int rl = (int)(rg - r0);
      if (rl < 0 || rl >= nr) return -1;
      int64_t ia = g.a0 + rg, ib = g.b0 + col;
      // self pairs: an entry below the diagonal was evaluated with the
      // column's box as P (the lower index), so the row's box is Q there
      const bool swapped = SELF && rg > col;
      if (swapped) {
        const int64_t t = ia;
        ia = ib;
        ib = t;
      }
      const int n1 = FIXED ? K : poly_count(m.a.nv, ia, m.a.kmax);
      const int n2 = FIXED ? K : poly_count(m.b.nv, ib, m.b.kmax);
      Poly<K> P, Q;
      load_poly<K, FIXED>(m.a.xy, ia, m.a.kmax, m.a.vec4, n1, P);
      load_poly<K, FIXED>(m.b.xy, ib, m.b.kmax, m.b.vec4, n2, Q);
      // self pairs: entries (i, k) and (k, i) are one unordered pair with
      // one structure, so the row's box takes its role's gradient of that
      // pair weighted by both entries' upstream gradients
      float gw = m.grad[pid];
      if constexpr (SELF) gw += m.grad[g.out0 + col * g.nb + rg];
      float lo1 = 0.f, hi1 = 0.f, lo2 = 0.f, hi2 = 0.f;
      if (Z3) {
        lo1 = m.a.zlo[ia];
        hi1 = m.a.zhi[ia];
        lo2 = m.b.zlo[ib];
        hi2 = m.b.zhi[ib];
      }
      float2 gP[K], gQ[K], gz1, gz2;
      bool thin;
      pair_backward<K, FIXED, Z3, BLOCK>(P, n1, Q, n2, gw, nx, codes, lo1, hi1, lo2, hi2,
                                         s_v + tid, s_g + tid, s_tab, gP, gQ, gz1, gz2, thin);
      if (thin) {  // rare: the gradient again in fp64, from the polygons reloaded
        load_poly<K, FIXED>(m.a.xy, opaque(ia), m.a.kmax, m.a.vec4, n1, P);
        load_poly<K, FIXED>(m.b.xy, opaque(ib), m.b.kmax, m.b.vec4, n2, Q);
        stage_pair<K, BLOCK>(s_v + tid, P, Q);
        pair_backward64<K, FIXED, Z3, BLOCK>(n1, n2, gw, nx, codes, lo1, hi1, lo2, hi2,
                                             s_v + tid, s_g + tid, gP, gQ, gz1, gz2);
      }
      const int nr_own = swapped ? n2 : n1;  // the row box's vertex count
#pragma unroll
      for (int k = 0; k < K; ++k) {
        const bool own = FIXED || k < nr_own;  // padded slots: 0
        gv[k] = own ? (swapped ? gQ[k] : gP[k]) : make_float2(0.f, 0.f);
      }
      if constexpr (Z3) gv[K] = swapped ? gz2 : gz1;
      if constexpr (!SELF) stage_column<K, BLOCK>(s_v + tid, gQ, gz2, ib, n2);
      return rl;
    };
    for (int64_t e0 = e_begin + 64 * part; e0 < e_end; e0 += 64 * parts) {  // uniform: every lane sums
      float2 gv[H];  // read only where rl >= 0
      const int rl = entry(e0 + lane, gv);
      if constexpr (!SELF)
        add_columns<K, FIXED, Z3, BLOCK>(__ballot(rl >= 0), stage, m.gb_xy, m.b.kmax, m.gb_z);
      step_row_sums<H, BLOCK>(rl, gv, stage, acc);
    }
    if constexpr (SPLIT) {  // the wavefronts' sums, in their order; one group a workgroup
#pragma unroll
      for (int j = 0; j < NACC; ++j) s_g[j * BLOCK + tid] = acc[j];
      __syncthreads();
      if (wave != 0) break;
#pragma unroll
      for (int w = 1; w < WAVES; ++w) {
#pragma unroll
        for (int j = 0; j < NACC; ++j) {
          const float2 v = s_g[j * BLOCK + w * 64 + lane];
          acc[j].x += v.x;
          acc[j].y += v.y;
        }
      }
    }
    // each row of a belongs to exactly one row group: plain stores
#pragma unroll
    for (int j = 0; j < NACC; ++j) {
      const int c = lane + 64 * j;
      const int r = c / H, h = c - r * H;
      if (r < nr) {
        const int64_t ia = g.a0 + r0 + r;
        if (h < K) {
          if (h < kx) {
            m.ga_xy[(ia * kx + h) * 2] = acc[j].x;
            m.ga_xy[(ia * kx + h) * 2 + 1] = acc[j].y;
          }
        } else if (Z3) {
          m.ga_z[ia * 2] = acc[j].x;
          m.ga_z[ia * 2 + 1] = acc[j].y;
        }
      }
    }
  }
}

namespace {

template <bool B>
using Bool = std::integral_constant<bool, B>;

// Calls f(K, FIXED, Z3) with compile-time constants.
template <typename F>
void dispatch(int K, bool fixed, bool z3, F&& f) {
  auto go = [&](auto k, auto fx) {
    if (z3) f(k, fx, Bool<true>{}); else f(k, fx, Bool<false>{});
  };
  if (K == 4) {
    if (fixed) go(std::integral_constant<int, 4>{}, Bool<true>{});
    else go(std::integral_constant<int, 4>{}, Bool<false>{});
  } else {
    if (fixed) go(std::integral_constant<int, 8>{}, Bool<true>{});
    else go(std::integral_constant<int, 8>{}, Bool<false>{});
  }
}

bool valid_saved(const dgal_saved* s) {
  return s != nullptr && s->pair_id && s->nx && s->xflags && s->count && s->capacity >= 0 &&
         s->tile_start && s->tile_count && s->tile_mask && s->tile_capacity >= 0;
}

void zero(float* p, int64_t n, hipStream_t stream, Profiler* prof) {
  if (p != nullptr && n > 0) {
    const int64_t blocks = (n + 255) / 256;
    prof_begin(prof, stream);
    hipLaunchKernelGGL(k_fill_zero, dim3((unsigned)(blocks > 4096 ? 4096 : blocks)), dim3(256), 0,
                       stream, p, n);
    prof_end(prof, "k_fill_zero", stream);
  }
}

// Common validation of the matrix shapes; fills the segment arguments.
int check_shapes(dgal_polys a, dgal_polys b, const int64_t* a_off, const int64_t* b_off,
                 const int64_t* out_off, int nseg, int self_pairs, int64_t out_size,
                 const dgal_saved* saved, SegArgs& sa) {
  if (!valid_polys(a) || !valid_polys(b) || out_size < 0) return DGAL_EINVAL;
  if ((a.zlo == nullptr) != (b.zlo == nullptr)) return DGAL_EINVAL;
  const bool segmented = a_off != nullptr;
  if (segmented != (b_off != nullptr) || segmented != (out_off != nullptr)) return DGAL_EINVAL;
  if (segmented && (nseg < 1 || nseg > kMaxSeg)) return DGAL_EINVAL;
  if (self_pairs && !same_polys(a, b)) return DGAL_EINVAL;
  if (!segmented && (b.count >= (1 << 24) ||
                     (a.count > 0 && b.count > 0 && out_size / a.count < b.count)))
    return DGAL_EINVAL;
  if (!valid_saved(saved)) return DGAL_EINVAL;
  if (saved->tile_capacity > kScanTotals * (int64_t)kScanChunk) return DGAL_EINVAL;
  sa.a_off = a_off;
  sa.b_off = b_off;
  sa.out_off = out_off;
  sa.nseg = segmented ? nseg : 1;
  sa.a_count = a.count;
  sa.b_count = b.count;
  sa.out_size = out_size;
  sa.self_pairs = self_pairs;
  sa.tile_prefix = nullptr;
  sa.group_prefix = nullptr;
  sa.rows_log2 = 3;
  return DGAL_OK;
}

int64_t ceil_div(int64_t x, int64_t y) { return (x + y - 1) / y; }

}  // namespace

int matrix_forward(const CtxView& ctx, dgal_polys a, dgal_polys b, const int64_t* a_off,
                   const int64_t* b_off, const int64_t* out_off, int nseg, int self_pairs,
                   float* iou, int64_t out_size, dgal_saved* saved, hipStream_t stream,
                   const LaunchShape& shape) {
  SegArgs sa;
  const int st = check_shapes(a, b, a_off, b_off, out_off, nseg, self_pairs, out_size, saved, sa);
  if (st != DGAL_OK) return st;
  if (out_size > 0 && iou == nullptr) return DGAL_EINVAL;
  // the tile shape: the launch shape's, else the caller's, else the default
  const int R = shape.tile_rows > 0 ? shape.tile_rows
                : (saved->tile_rows > 0 ? saved->tile_rows : DGAL_TILE_ROWS_DEFAULT);
  sa.rows_log2 = tile_rows_log2(R);
  if (sa.rows_log2 < 0) return DGAL_EINVAL;
  saved->tile_rows = R;
  DeviceGuard dg(ctx.device);
  if (!dg.ok) return DGAL_EHIP;
  const int K = reg_k(a.kmax, b.kmax);
  const bool segmented = a_off != nullptr;
  int64_t single_tiles = 0;
  int64_t* pre = nullptr;
  if (segmented) {
    // in the caller's saved state when it has room, for the backward
    pre = saved->seg_prefix != nullptr ? saved->seg_prefix : ctx.prefix;
    sa.tile_prefix = pre;
    sa.group_prefix = pre + (kMaxSeg + 1);
  } else {
    if (a.count == 0 || b.count == 0) return hipGetLastError() == hipSuccess ? DGAL_OK : DGAL_EHIP;
    single_tiles = ceil_div(a.count, R) * ceil_div(b.count, kTilePairs / R);
  }
  CullArgs c;
  c.seg = sa;
  c.a = poly_args(a, K);
  c.b = poly_args(b, K);
  c.tile_count = saved->tile_count;
  c.tile_capacity = saved->tile_capacity;
  c.tile_mask = saved->tile_mask;
  c.tile_prefix = pre;
  c.group_prefix = segmented ? pre + (kMaxSeg + 1) : nullptr;
  c.err = ctx.err;
  // up to a 256-row unit a CU (4096 x 4096; of segments the output's size tells),
  // units of 64 rows whose words the wavefronts share: more workgroups, each a
  // quarter of the tests, where the chip would be idle and the busiest unit is
  // the pass.  256 / 64 rows, the whole forward in us: 2000 x 301 16.8 / 14.0,
  // in a crowd 23.8 / 18.4; 4096 x 4096 30.6 / 30.1, in grid order 32.7 / 30.2;
  // 8 scenes of 50..2000 33.2 / 31.5.  Past it the columns' bins, made four times
  // as often, cost more: 5000 x 5000 36.9 / 38.2, 64 scenes 114 / 132.
  const bool words = (segmented ? out_size : a.count * b.count) <= (int64_t)ctx.cus * 65536;
  // the units' workgroups; with segments, whose sizes are on the device, they
  // walk the units in grid strides
  int64_t cull_grid = (int64_t)ctx.cus * (shape.cull_mult > 0 ? shape.cull_mult : 8);
  if (segmented) {
    c.single_units = 0;
    cull_grid = std::max<int64_t>(1, std::min(cull_grid, saved->tile_capacity));
  } else {
    c.single_units = ceil_div(a.count, unit_rows_of(words)) * ceil_div(b.count, kTilePairs / R);
    cull_grid = std::min(cull_grid, c.single_units);
  }
  ListArgs li;
  li.seg = sa;
  li.single_tiles = single_tiles;
  li.iou = iou;
  li.tile_capacity = saved->tile_capacity;
  li.tile_count = saved->tile_count;
  li.totals = nullptr;
  li.tile_mask = saved->tile_mask;
  li.tile_start = saved->tile_start;
  li.pair_id = saved->pair_id;
  li.capacity = saved->capacity;
  li.count = saved->count;
  li.err = ctx.err;
  ExactArgs x;
  x.seg = sa;
  x.a = c.a;
  x.b = c.b;
  x.iou = iou;
  x.pair_id = saved->pair_id;
  x.s_nx = saved->nx;
  x.s_flags = saved->xflags;
  x.capacity = saved->capacity;
  x.count = saved->count;
  x.cap = a.kmax + b.kmax;
  x.flags_vec = x.cap == 2 * K && aligned(saved->xflags, (uintptr_t)x.cap);
  x.err = ctx.err;
  x.stats = ctx.stats;
  x.tile_start = saved->tile_start;
  x.tile_count = saved->tile_count;
  x.tile_capacity = saved->tile_capacity;
  x.single_tiles = single_tiles;
  const int exact_grid = ctx.cus * (shape.exact_mult > 0 ? shape.exact_mult : 8);
  const bool fixed = a.nv == nullptr && b.nv == nullptr && a.kmax == K && b.kmax == K &&
                     aligned(a.xy, 16) && aligned(b.xy, 16);
  dispatch(K, fixed, a.zlo != nullptr, [&](auto k, auto fx, auto z) {
    constexpr int KK = decltype(k)::value;
    constexpr bool FX = decltype(fx)::value, ZZ = decltype(z)::value;
    prof_begin(ctx.prof, stream);
    const dim3 cg((unsigned)cull_grid), cb(kCullBlock);
    auto cull = [&](auto rows) {
      constexpr int RR = decltype(rows)::value;
      if (words) hipLaunchKernelGGL((k_matrix_cull<KK, FX, ZZ, RR, true>), cg, cb, 0, stream, c);
      else hipLaunchKernelGGL((k_matrix_cull<KK, FX, ZZ, RR, false>), cg, cb, 0, stream, c);
    };
    if (R == 4) cull(std::integral_constant<int, 4>{});
    else if (R == 16) cull(std::integral_constant<int, 16>{});
    else cull(std::integral_constant<int, 8>{});
    prof_end(ctx.prof, "k_matrix_cull", stream);
    if (saved->tile_capacity > kListDirect) {
      const int64_t chunks = ceil_div(saved->tile_capacity, kScanChunk);
      prof_begin(ctx.prof, stream);
      hipLaunchKernelGGL(k_scan_totals, dim3((unsigned)chunks), dim3(kScanBlock), 0, stream,
                         sa.tile_prefix, sa.nseg, single_tiles, saved->tile_capacity,
                         saved->tile_count, ctx.scan);
      prof_end(ctx.prof, "k_scan_totals", stream);
      li.totals = ctx.scan;
    }
    // the list's workgroups first, then the fill's, a step each up to the
    // launch's limit on threads
    // (8 tiles are a workgroup's step: 300 x 300 boxes that mostly overlap take
    // 26 us with twice as many, 21.5 so)
    li.list_blocks = std::max<int64_t>(
        1, std::min<int64_t>((int64_t)ctx.cus * 2, ceil_div(saved->tile_capacity, 8)));
    const int64_t fill = ceil_div((segmented ? out_size : a.count * b.count) + 3, kFillStep);
    prof_begin(ctx.prof, stream);
    hipLaunchKernelGGL(k_matrix_list,
                       dim3((unsigned)(li.list_blocks + std::min<int64_t>(1 << 23, fill))),
                       dim3(kListBlock), 0, stream, li);
    prof_end(ctx.prof, "k_matrix_list", stream);
    prof_begin(ctx.prof, stream);
    hipLaunchKernelGGL((k_matrix_exact<KK, FX, ZZ>), dim3(exact_grid), dim3(kExactBlock), 0,
                       stream, x);
    prof_end(ctx.prof, "k_matrix_exact", stream);
  });
  return hipGetLastError() == hipSuccess ? DGAL_OK : DGAL_EHIP;
}

int matrix_backward(const CtxView& ctx, dgal_polys a, dgal_polys b, const int64_t* a_off,
                    const int64_t* b_off, const int64_t* out_off, int nseg, int self_pairs,
                    const float* grad_iou, int64_t out_size, const dgal_saved* saved,
                    float* grad_a_xy, float* grad_b_xy, float* grad_a_z, float* grad_b_z,
                    hipStream_t stream, const LaunchShape& shape) {
  SegArgs sa;
  const int st = check_shapes(a, b, a_off, b_off, out_off, nseg, self_pairs, out_size, saved, sa);
  if (st != DGAL_OK) return st;
  const bool z3 = a.zlo != nullptr;
  if (grad_iou == nullptr || grad_a_xy == nullptr) return DGAL_EINVAL;
  if (self_pairs ? (grad_b_xy != nullptr || grad_b_z != nullptr) : (grad_b_xy == nullptr))
    return DGAL_EINVAL;
  if (z3 != (grad_a_z != nullptr)) return DGAL_EINVAL;
  if (!self_pairs && z3 != (grad_b_z != nullptr)) return DGAL_EINVAL;
  sa.rows_log2 = tile_rows_log2(saved->tile_rows);  // the shape the forward recorded
  if (sa.rows_log2 < 0) return DGAL_EINVAL;
  DeviceGuard dg(ctx.device);
  if (!dg.ok) return DGAL_EHIP;
  const int K = reg_k(a.kmax, b.kmax);
  const bool segmented = a_off != nullptr;
  // every row of a is written by its row group, or zeroed by the kernel when
  // no row group holds it (segmented); without segments an empty b leaves no
  // row group at all.  Columns of a second set take atomic adds: zeroed
  // first.
  if (!segmented && b.count == 0) {
    zero(grad_a_xy, a.count * a.kmax * 2, stream, ctx.prof);
    if (z3) zero(grad_a_z, a.count * 2, stream, ctx.prof);
  }
  if (!self_pairs) {
    zero(grad_b_xy, b.count * b.kmax * 2, stream, ctx.prof);
    if (z3) zero(grad_b_z, b.count * 2, stream, ctx.prof);
  }
  int64_t single_groups = 0;
  if (segmented) {
    if (saved->seg_prefix != nullptr) {  // the forward's, kept with its work list
      sa.tile_prefix = saved->seg_prefix;
      sa.group_prefix = saved->seg_prefix + (kMaxSeg + 1);
    } else {
      // recomputed: another matrix call may have used the workspace since the forward
      sa.tile_prefix = ctx.prefix;
      sa.group_prefix = ctx.prefix + (kMaxSeg + 1);
      prof_begin(ctx.prof, stream);
      hipLaunchKernelGGL(k_seg_prep, dim3(1), dim3(256), 0, stream, sa, ctx.err, ctx.prefix,
                         ctx.prefix + (kMaxSeg + 1));
      prof_end(ctx.prof, "k_seg_prep", stream);
    }
  } else {
    if (a.count == 0 || b.count == 0) return hipGetLastError() == hipSuccess ? DGAL_OK : DGAL_EHIP;
    single_groups = ceil_div(a.count, kGroupRows);
  }
  BwdArgs m;
  m.seg = sa;
  m.a = poly_args(a, K);
  m.b = poly_args(b, K);
  m.single_groups = single_groups;
  m.grad = grad_iou;
  m.pair_id = saved->pair_id;
  m.s_nx = saved->nx;
  m.s_flags = saved->xflags;
  m.flags_vec = a.kmax + b.kmax == 2 * reg_k(a.kmax, b.kmax) &&
                aligned(saved->xflags, (uintptr_t)(a.kmax + b.kmax));
  m.capacity = saved->capacity;
  m.tile_start = saved->tile_start;
  m.tile_count = saved->tile_count;
  m.tile_capacity = saved->tile_capacity;
  m.cap = a.kmax + b.kmax;
  m.ga_xy = grad_a_xy;
  m.gb_xy = grad_b_xy;
  m.ga_z = grad_a_z;
  m.gb_z = grad_b_z;
  const bool fixed = a.nv == nullptr && b.nv == nullptr && a.kmax == K && b.kmax == K &&
                     aligned(a.xy, 16) && aligned(b.xy, 16);
  dispatch(K, fixed, z3, [&](auto k, auto fx, auto z) {
    constexpr int KK = decltype(k)::value;
    constexpr bool FX = decltype(fx)::value, ZZ = decltype(z)::value;
    int64_t grid = (int64_t)ctx.cus * (shape.bwd_mult > 0 ? shape.bwd_mult : 8);
    const bool split = matrix_bwd_split(ctx, segmented, K, a.count, b.count);
    if (split)
      grid = single_groups;
    else if (!segmented)
      grid = std::min(grid, ceil_div(single_groups, bwd_block<KK>() / 64));
    prof_begin(ctx.prof, stream);
    auto go = [&](auto self, auto split) {
      hipLaunchKernelGGL((k_matrix_bwd<KK, FX, ZZ, decltype(self)::value, decltype(split)::value>),
                         dim3((unsigned)grid), dim3(bwd_block<KK>()), 0, stream, m);
    };
    if (self_pairs && split) go(Bool<true>{}, Bool<true>{});
    else if (self_pairs) go(Bool<true>{}, Bool<false>{});
    else if (split) go(Bool<false>{}, Bool<true>{});
    else go(Bool<false>{}, Bool<false>{});
    prof_end(ctx.prof, "k_matrix_bwd", stream);
  });
  return hipGetLastError() == hipSuccess ? DGAL_OK : DGAL_EHIP;
}


// ---- scratch of the allocation-free forward (dgal_iou_matrix_noalloc) ----
// The work list, tile state, segment prefixes and scan totals that
// dgal_iou_matrix takes from the caller's dgal_saved and the context live
// here instead, in one static device array per GPU (allocated when the
// library's code object is loaded on that GPU, held until the process ends).
// Every call on a GPU shares its array: two such calls that overlap on one
// GPU race.  Nothing in it must start at zero (the forward writes every
// field it later reads, including the survivor count).
constexpr int64_t kNaTiles = DGAL_NOALLOC_MAX_TILES;
constexpr int64_t kNaPairs = DGAL_NOALLOC_MAX_PAIRS;
constexpr int64_t kNaFlags = 16;  // codes per entry: kmax_a + kmax_b <= 16
constexpr int64_t align256(int64_t v) { return (v + 255) & ~(int64_t)255; }
constexpr int64_t kNaPrefix = 0;  // int64 [2][DGAL_MAX_SEGMENTS + 1]
constexpr int64_t kNaScan = align256(kNaPrefix + 8 * 2 * (DGAL_MAX_SEGMENTS + 1));
constexpr int64_t kNaCount = align256(kNaScan + 8 * kScanTotals);
constexpr int64_t kNaTileStart = align256(kNaCount + 8);
constexpr int64_t kNaTileCount = align256(kNaTileStart + 8 * kNaTiles);
constexpr int64_t kNaTileMask = align256(kNaTileCount + 4 * kNaTiles);
constexpr int64_t kNaPairId = align256(kNaTileMask + 8 * kMaskWords * kNaTiles);
constexpr int64_t kNaNx = align256(kNaPairId + 8 * kNaPairs);
constexpr int64_t kNaXflags = align256(kNaNx + kNaPairs);
constexpr int64_t kNaBytes = align256(kNaXflags + kNaFlags * kNaPairs);
static_assert(kNaBytes == DGAL_NOALLOC_SCRATCH_BYTES, "scratch size stated in dgal.h");

static __device__ __align__(256) unsigned char scratch[kNaBytes];

namespace {
constexpr int kNaDevices = 64;
std::mutex na_mu;
void* na_ptr[kNaDevices] = {};  // device address of `scratch` per GPU
}  // namespace

// Takes the device address of `scratch` on `device` (which must be current)
// once; later calls for the same device return at once.
int matrix_scratch_init(int device) {
  if (device < 0 || device >= kNaDevices) return DGAL_EINVAL;
  std::lock_guard<std::mutex> lock(na_mu);
  if (na_ptr[device] != nullptr) return DGAL_OK;
  void* ptr = nullptr;
  if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || ptr == nullptr)
    return DGAL_EHIP;
  na_ptr[device] = ptr;
  return DGAL_OK;
}

int matrix_forward_noalloc(const CtxView& ctx, dgal_polys a, dgal_polys b, const int64_t* a_off,
                           const int64_t* b_off, const int64_t* out_off, int nseg,
                           int self_pairs, float* iou, int64_t out_size, hipStream_t stream,
                           const LaunchShape& shape) {
  void* base_v = nullptr;
  if (ctx.device >= 0 && ctx.device < kNaDevices) {
    std::lock_guard<std::mutex> lock(na_mu);
    base_v = na_ptr[ctx.device];
  }
  if (base_v == nullptr) return DGAL_EHIP;  // the context did not set this device up
  // one block: its tile count is known here, and a block past the scratch's
  // tiles is refused before anything is enqueued
  const int R = shape.tile_rows > 0 ? shape.tile_rows : DGAL_TILE_ROWS_DEFAULT;
  if (tile_rows_log2(R) < 0) return DGAL_EINVAL;
  if (a_off == nullptr && a.count > 0 && b.count > 0 &&
      ceil_div(a.count, R) > kNaTiles / ceil_div(b.count, kTilePairs / R))
    return DGAL_ECAPACITY;
  unsigned char* base = static_cast<unsigned char*>(base_v);
  dgal_saved sv;
  sv.pair_id = reinterpret_cast<int64_t*>(base + kNaPairId);
  sv.nx = base + kNaNx;
  sv.xflags = base + kNaXflags;
  sv.capacity = kNaPairs;
  sv.count = reinterpret_cast<int64_t*>(base + kNaCount);
  sv.tile_start = reinterpret_cast<int64_t*>(base + kNaTileStart);
  sv.tile_count = reinterpret_cast<int32_t*>(base + kNaTileCount);
  sv.tile_capacity = kNaTiles;
  sv.tile_mask = reinterpret_cast<uint64_t*>(base + kNaTileMask);
  sv.tile_rows = R;
  sv.seg_prefix = nullptr;  // the scratch's own prefixes
  CtxView v = ctx;
  v.prefix = reinterpret_cast<int64_t*>(base + kNaPrefix);
  v.scan = reinterpret_cast<int64_t*>(base + kNaScan);
  return matrix_forward(v, a, b, a_off, b_off, out_off, nseg, self_pairs, iou, out_size, &sv,
                        stream, shape);
}

}  // namespace dgal
