// Tile lists by counting and one small sort per cell of 2x2 tiles (Sec. III-A depth order,
// Sec. III-D.2 footprint tiles).
//
// Input: per (view, Gaussian) pair its depth and the tiles it reaches. Output: every tile's
// Gaussians by (depth, index), consecutive in one array in tile order, and the tiles' ranges:
//   k_cell_count    each block counts its pairs' entries per cell, and the hits of the cell's
//                   four tiles, in LDS -> its row of the view's matrices;
//   k_cell_colscan  exclusive prefix of every cell's entries over the rows, and the totals;
//   k_cell_offsets  exclusive scans of the totals: tile ranges, cell starts, the instance
//                   count, overflow, and the cells past the small block size;
//   k_cell_place    each block walks its pairs again and writes one entry (depth, Gaussian,
//                   which of the four tiles) per cell it reaches at the cell's next position,
//                   in any order within the block;
//   k_cell_sort_small, k_cell_sort_large
//                   one block per cell orders its entries in LDS and deals them out to its
//                   tiles' lists by ballots (two sizes of block); cells of more than kSortMost
//                   entries are ordered in chunks, which k_cell_rank or k_cell_merge deals out.
// (depth, Gaussian) is unique in a cell, so the lists do not depend on the order of arrival.
//
// Why cells: what bounds the placement is not its bytes but the scattered writes, which L2
// writes back as partial lines (one 8-B entry per hit: 272 MB written for 55 MB of entries at
// 6.9 M hits, 97 us; one per cell: 114 MB, 44 us then), and a Gaussian reaches two to three times
// fewer cells than tiles, which the sort gains as well.
//
// Measured against the path it replaced where it applies (a depth sort of the pairs by four
// radix passes, a scan of the counts in that order, an emission, two radix passes by tile id,
// the ranges), in us: 1M Gaussians at 1280x720 (6.9 M instances) 257 -> 126; eight views of 1M
// (41.6 M) 1416 -> 623; 3M at 1920x1200 (35.9 M) 917 -> 526; a street map of 520k with a long
// horizon (0.7 M) 149 -> 89; 10k at 256x192 (17.8 k) 99 -> 29, of which most were launches
// (20 -> 6). At 1M the counting takes 27, the column and total scans 18, the placement 33 and
// the sort 39. Counting and placing issue VALU work for more than half of their time; the sort
// of a cell is a chain of LDS steps and barriers.
//
// The LDS counters bound the cells of a view (tile_lists_fit); larger images take the radix
// path (binning.hip).
#include "blend_split.h"
#include "gs_common.h"
#include "kernels.h"

namespace gs {

constexpr int kTlThreads = 512;          // of the counting and placing blocks
constexpr int kTlMaxCells = 13000;       // 12 B of counters each: within a CU's 160 KiB of LDS
constexpr int kTlMaxPairs = 32768;       // of one block: its hits per tile are counted in 16 bits
constexpr int kTlMaskBits = 4;           // entry: depth bits << 32 | Gaussian << 4 | tiles
constexpr int64_t kTlMaxId = int64_t(1) << (32 - kTlMaskBits);

// Cells are ordered by blocks of two sizes: up to 4096 and 16384 entries (four and one of them
// fit a CU's LDS). Larger cells are ordered in chunks of at most the larger size; the merge
// holds a cell's chunks, up to four per lane of a block, in LDS, which bounds the Gaussians of
// a map (a cell holds each once): larger maps take the radix path.
template <bool LARGE>
struct SortShape {
  static constexpr int cap = 4096, threads = 512;
};
template <>
struct SortShape<true> {
  static constexpr int cap = 16384, threads = 1024;
};
constexpr int kSortSmall = SortShape<false>::cap, kSortMost = SortShape<true>::cap;
constexpr int kMostChunks = 4096;
constexpr int64_t kTlMostGaussians = (int64_t)kMostChunks * kSortMost;
__device__ __forceinline__ int sort_chunks(uint32_t n) { return (int)((n + kSortMost - 1) / kSortMost); }

__host__ __device__ __forceinline__ int cells_of(int tiles) { return (tiles + 1) >> 1; }
__device__ __forceinline__ int view_cells(const ViewDev& V) { return cells_of(V.tiles_x) * cells_of(V.tiles_y); }

// Cells of the views, all views together; first cell of each view in `base` if given.
static int64_t cells_total(const ViewsArg& va, int32_t* base = nullptr) {
  int64_t c = 0;
  for (int v = 0; v < va.n; ++v) {
    if (base) base[v] = (int32_t)c;
    c += (int64_t)cells_of(va.v[v].tiles_x) * cells_of(va.v[v].tiles_y);
  }
  return c;
}

static int max_cells(const ViewsArg& va) {
  int c = 1;
  for (int v = 0; v < va.n; ++v) c = std::max(c, cells_of(va.v[v].tiles_x) * cells_of(va.v[v].tiles_y));
  return c;
}

// A map of far more Gaussians than the images have room for fills few cells with many chunks
// each; the radix path's time does not depend on the cells. The binning of a render over 64x48
// (four cells), here and there, in us: 50000 per cell 97 and 113, 125000 138 and 123, 250000
// 151 and 150, 1M 395 and 358. Below the line, but with all of them in one cell of 1280x720:
// 200k 138 and 150, 1M 216 and 220, 2M 298 and 309, 4M 567 and 473.
constexpr int64_t kTlMostPerCell = 65536;

bool tile_lists_fit(const ViewsArg& va, int64_t N, int64_t max_instances) {
  if (va.n * N > kTlMostPerCell * cells_total(va)) return false;
  for (int v = 0; v < va.n; ++v)
    if ((int64_t)cells_of(va.v[v].tiles_x) * cells_of(va.v[v].tiles_y) > kTlMaxCells) return false;
  return N <= kTlMostGaussians && max_instances < kTlMaxId;
}

// How the views' pairs fall to the blocks: view v's are shared by blocks [block[v],
// block[v + 1]), each with a matrix row of the view's cells from word `matrix[v]` on; its
// cells are numbered from cell[v].
struct CellBase {
  int32_t cell[kMaxViews];
  int32_t block[kMaxViews + 1];
  int64_t matrix[kMaxViews];
};

// Blocks of 512 lanes: about 1024 pairs each (512 to 4096 blocks), since blocks of more pairs
// end unevenly and spread their writes (3M Gaussians, 1920x1200: count and place 180 and 305 us
// with 512 blocks, 113 and 152 with 2929; 8 x 1M at 1280x720: 137 and 300 with 1024, 109 and
// 222 with 4096), while a block of fewer writes and reads its matrix row for little; but no
// more than make kTlMatrix matrix entries (3M at 3840x2160: a render of 4211 us without this
// bound, 3526 with it). Shared out by the views' cells (a view's entries grow with its size)
// plus an even part (its pairs do not), at least 256 pairs each. A view's count is a multiple
// of eight (xcd_block).
constexpr int64_t kTlMatrix = int64_t(8) << 20;
static CellBase cell_base(const ViewsArg& va, int32_t N) {
  CellBase b{};
  const int64_t cells = cells_total(va, b.cell), most_rows = kTlMatrix * va.n / cells,
                grid = std::clamp<int64_t>((int64_t)va.n * N / 1024, 512, std::clamp<int64_t>(most_rows, 512, 4096));
  const int64_t fewest = ((int64_t)N + kTlMaxPairs - 1) / kTlMaxPairs, most = std::max<int64_t>(1, ((int64_t)N + 255) / 256);
  int64_t words = 0;
  for (int v = 0; v < va.n; ++v) {
    const int64_t nc = (int64_t)cells_of(va.v[v].tiles_x) * cells_of(va.v[v].tiles_y);
    const int64_t share = grid * (nc * va.n + cells) / (2 * cells * va.n);
    int64_t G = std::min(std::max(share, fewest), most);
    if (va.n > 1) G = (G + 7) & ~int64_t(7);
    b.block[v + 1] = b.block[v] + (int32_t)G;
    b.matrix[v] = words;
    words += G * nc;
  }
  return b;
}
static int64_t matrix_words(const ViewsArg& va, const CellBase& b) {
  const ViewDev& V = va.v[va.n - 1];
  return b.matrix[va.n - 1] +
         (int64_t)(b.block[va.n] - b.block[va.n - 1]) * cells_of(V.tiles_x) * cells_of(V.tiles_y);
}

// The block's view, its number in the view and the view's blocks.
__device__ __forceinline__ int view_of_block(const CellBase& cb, int n_views, int& g, int& G) {
  int v = 0;
  for (int k = 1; k < n_views; ++k)
    if ((int)blockIdx.x >= cb.block[k]) v = k;
  G = cb.block[v + 1] - cb.block[v];
  g = xcd_block((int)blockIdx.x - cb.block[v], G);
  return v;
}

// Pair i of block g of G (from its first on, i < block_pairs): runs of kTlRun pairs go round
// the blocks, so that Gaussians that lie side by side in the map (a depth image's, a street's
// near ones with hundreds of cells each) spread over all of them.
constexpr int kTlRun = 16;
__device__ __forceinline__ int pair_of(int i, int g, int G) { return ((i / kTlRun) * G + g) * kTlRun + i % kTlRun; }
__device__ __forceinline__ int block_pairs(int N, int g, int G) {
  const int runs = (N + kTlRun - 1) / kTlRun;
  return g < runs ? ((runs - 1 - g) / G + 1) * kTlRun : 0;  // (the last may reach past N)
}

// Workspace: per cell and block the packed hits (8 B) and the entries (4 B); per cell its
// entries and its first one (one more at the end), per tile its hits; and the work items of
// the larger sorting blocks: every cell past the small size with its first chunk (or whole),
// and, by the instance capacity, the chunks after a cell's first.
enum { kItems, kExtra, kTlCounts };  // TlSpace::count
struct TlSpace {
  uint64_t* hits;
  uint32_t* entries;
  uint32_t* sizes;
  uint32_t* start;
  uint32_t* totals;
  uint4* items;      // (cell, chunk, the cell's first entry, its entries), in any order
  uint32_t* lists;   // per cell, where its four tiles' lists start
  uint32_t* count;   // items; chunks after a cell's first
};
int64_t tile_space_bytes(const ViewsArg& va, int32_t N) {
  const int64_t c = cells_total(va), m = matrix_words(va, cell_base(va, N));
  return 12 * m + 16 * (2 * c) + 4 * (2 * c + 1 + va.total_tiles + kTlCounts) + 256;
}
// Chunks after a cell's first: n entries of a cell have less than n / kSortMost, and the
// entries of all cells are at most the instances.
static int64_t most_extra(int64_t instances) { return instances / kSortMost + 1; }
int64_t tile_extra_bytes(int64_t instances) { return 16 * most_extra(instances); }
static TlSpace tl_space(void* ws, const ViewsArg& va, const CellBase& cb) {
  const int64_t c = cells_total(va), m = matrix_words(va, cb);
  TlSpace t;
  t.items = (uint4*)ws;
  t.lists = (uint32_t*)(t.items + c);
  t.hits = (uint64_t*)(t.lists + 4 * c);
  t.entries = (uint32_t*)(t.hits + m);
  t.sizes = t.entries + m;
  t.start = t.sizes + c;
  t.totals = t.start + c + 1;
  t.count = t.totals + va.total_tiles;
  return t;
}

// Tile rectangle of a pair's 16-B word: x0 | y0 << 16, x1 | y1 << 16, 64-bit hit mask.
struct PairRect {
  int x0, y0, rw, rh;
};
__device__ __forceinline__ PairRect pair_rect(uint32_t a, uint32_t b) {
  PairRect r;
  r.x0 = (int)(a & 0xffffu);
  r.y0 = (int)(a >> 16);
  r.rw = (int)(b & 0xffffu) - r.x0 + 1;
  r.rh = (int)(b >> 16) - r.y0 + 1;
  return r;
}

// Calls entry(cell, tiles, lane of the pair, hits of the pair in its earlier cells, the pair's
// d and e) once for every cell that one of the wave's 64 pairs reaches (q: the lane's pair
// word, zero without hits; rp: its record; d, e: values that travel with it). tiles: bit
// 2 row + column per tile of the cell. A pair's cells come in row-major order. HITS = false:
// the earlier cells' hits are not needed. `own_row`: 64 B of LDS of this wave.
//
// The cells of the rectangles of up to 64 tiles are laid end to end over the lanes, 64 a step,
// whatever the pairs' sizes (in index order a wave's largest pair has about ten times the
// mean). A lane's owner is the last pair that starts at or before it: the last start mark in
// the step, or the pair that holds the step's first cell. Larger rectangles are left to
// for_each_large_cell: the lanes that hold one are returned.
template <bool HITS, typename F>
__device__ __forceinline__ uint64_t for_each_cell(uint4 q, uint32_t d, uint32_t e, int cells_x, uint8_t* own_row,
                                                  F entry) {
  const int lane = threadIdx.x & 63;
  const uint64_t upto = ~0ull >> (63 - lane);
  const PairRect r = pair_rect(q.x, q.y);
  const bool large = r.rw * r.rh > 64;
  const int hits = large ? 0 : __popc(q.z) + __popc(q.w);
  const int ncw = ((r.x0 + r.rw - 1) >> 1) - (r.x0 >> 1) + 1, nch = ((r.y0 + r.rh - 1) >> 1) - (r.y0 >> 1) + 1;
  const int a = hits ? ncw * nch : 0;  // at most 34 (17 x 2: 32 x 2 tiles off both edges of a cell), 33 wide
  const int end = wave_scan(a);
  const int beg = end - a;
  const int hbeg = HITS ? wave_scan(hits) - hits : 0;
  const int total = __builtin_amdgcn_readlane(end, 63);
  int done = 0;  // hits of the steps before
  for (int base = 0; base < total; base += 64) {  // wave-uniform
    own_row[lane] = 0xff;
    wave_lds_sync();
    if (a > 0 && beg >= base && beg < base + 64) own_row[beg - base] = (uint8_t)lane;
    wave_lds_sync();
    const int mark = own_row[lane];
    const int first = __popcll(__ballot(end <= base));
    const uint64_t before = __ballot(mark != 0xff) & upto;
    const int own = before ? __shfl(mark, 63 - __clzll((long long)before), 64) : first;
    wave_lds_sync();  // the row is rewritten in the next step
    const uint32_t qx = __shfl(q.x, own), qy = __shfl(q.y, own), mlo = __shfl(q.z, own), mhi = __shfl(q.w, own);
    const int k = base + lane - __shfl(beg, own), ohb = HITS ? __shfl(hbeg, own) : 0;
    const uint32_t od = __shfl(d, own), oe = __shfl(e, own);
    const PairRect o = pair_rect(qx, qy);
    const int cx0 = o.x0 >> 1, cw = ((o.x0 + o.rw - 1) >> 1) - cx0 + 1;
    // row and column of cell k < 64 among cw <= 33: the quotient's fractional part is a
    // multiple of 1 / cw and k * rcp(cw) is within 64 x 2^-23 of k / cw, so adding 1 / 128
    // before truncating gives the exact quotient
    const int cr = (int)fmaf((float)k, __builtin_amdgcn_rcpf((float)cw), 1.0f / 128.0f);
    const int cx = cx0 + k - cr * cw, cy = (o.y0 >> 1) + cr;
    // the cell's tiles in the mask: columns dx, dx + 1 of rows dy, dy + 1 (-1: left of or above
    // the rectangle)
    const int dx = 2 * cx - o.x0, dy = 2 * cy - o.y0;
    const uint64_t mask = (uint64_t)mhi << 32 | mlo;
    const uint32_t cols = (dx >= 0 ? 1u : 0u) | (dx + 1 < o.rw ? 2u : 0u);
    uint32_t tiles = 0;
#pragma unroll
    for (int row = 0; row < 2; ++row) {
      const int y = dy + row, p = y * o.rw + dx;
      // (p = -1 only in row 0 of the rectangle, one column left of it)
      const uint32_t two = p >= 0 ? (uint32_t)(mask >> (p & 63)) & 3u : ((uint32_t)mask & 1u) << 1;
      if (y >= 0 && y < o.rh) tiles |= (two & cols) << (2 * row);
    }
    if (base + lane >= total) tiles = 0;
    const int n = __popc(tiles), run = HITS ? wave_scan(n) : 0;
    if (tiles) entry(cy * cells_x + cx, tiles, own, (uint32_t)(done + run - n - ohb), od, oe);
    if (HITS) done += __builtin_amdgcn_readlane(run, 63);
  }
  return __ballot(large);
}

// The cells of one pair with a rectangle of more than 64 tiles: the tile predicate is
// evaluated again, 16 cells a step, of which this wave takes steps s0, s0 + ds, ... (HITS: all
// of them). q, rp: the pair's word and record (the same in every lane); entry as above,
// without the lane.
template <bool HITS, typename F>
__device__ __forceinline__ void for_each_large_cell(uint4 q, const float4* __restrict__ rp, int cells_x, int s0, int ds,
                                                    F entry) {
  const int lane = threadIdx.x & 63;
  const PairRect r = pair_rect(q.x, q.y);
  const float4 r0 = rp[0];
  const float C = rp[1].x, thr = rp[2].w;
  const int cx0 = r.x0 >> 1, cy0 = r.y0 >> 1;
  const int cw = ((r.x0 + r.rw - 1) >> 1) - cx0 + 1, cells = cw * (((r.y0 + r.rh - 1) >> 1) - cy0 + 1);
  uint32_t seen = 0;
  for (int c0 = 16 * s0; c0 < cells; c0 += 16 * ds) {
    const int c = c0 + (lane >> 2);
    const int cy = cy0 + c / cw, cx = cx0 + c % cw;
    const int tx = 2 * cx + (lane & 1), ty = 2 * cy + ((lane >> 1) & 1);
    const bool h = c < cells && tx >= r.x0 && tx < r.x0 + r.rw && ty >= r.y0 && ty < r.y0 + r.rh &&
                   key_tile_hit(r0.x, r0.y, r0.z, r0.w, C, thr, tx, ty);
    const uint64_t m = __ballot(h);
    const uint32_t tiles = (uint32_t)(m >> (lane & 60)) & 15u;
    if ((lane & 3) == 0 && tiles)
      entry(cy * cells_x + cx, tiles, HITS ? seen + (uint32_t)__popcll(m & ((1ull << lane) - 1ull)) : 0u);
    if (HITS) seen += (uint32_t)__popcll(m);
  }
}

// The large pairs of a block, collected while its waves walk the others and shared out to all
// of them afterwards: a map's few near Gaussians cover hundreds of cells each and lie side by
// side in it. Where the wave that met them walked them alone and a block's pairs were a run of
// the map, count and place took 79 and 81 us at four views of 96k Gaussians (1477 such pairs)
// at 1575x1033 and 41 and 38 at 520k Gaussians of a street at 1280x720; now 19 and 19, 12 and
// 12. Both are needed: sharing alone left 86 and 89.
constexpr int kLargeMost = 128;
struct LargeList {
  uint32_t n;
  uint16_t pair[kLargeMost];  // their numbers in the block
};
// Puts the lanes' pairs of `larges` on the list; returns those that no longer fit.
__device__ __forceinline__ uint64_t keep_large(LargeList& L, uint64_t larges, int pair) {
  const int lane = threadIdx.x & 63;
  uint32_t at = 0;
  if (lane == 0) at = atomicAdd(&L.n, (uint32_t)__popcll(larges));
  at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at) + (uint32_t)__popcll(larges & ((1ull << lane) - 1ull));
  const bool mine = (larges >> lane) & 1ull;
  if (mine && at < (uint32_t)kLargeMost) L.pair[at] = (uint16_t)pair;
  return __ballot(mine && at >= (uint32_t)kLargeMost);
}

// Each block's row of both matrices.
__global__ void __launch_bounds__(kTlThreads) __attribute__((amdgpu_waves_per_eu(8)))
k_cell_count(const float4* __restrict__ rec, const uint4* __restrict__ pairs, int32_t N, ViewsArg va, CellBase cb,
             TlSpace ws) {
  extern __shared__ uint64_t s_cells[];
  __shared__ uint8_t s_own[kTlThreads];
  __shared__ LargeList s_large;
  int g, G;
  const int v = view_of_block(cb, va.n, g, G);
  const ViewDev& V = va.v[v];
  const int nc = view_cells(V), cells_x = cells_of(V.tiles_x);
  uint64_t* s_hits = s_cells;                       // [nc] four 16-bit counts
  uint32_t* s_entries = (uint32_t*)(s_cells + nc);  // [nc]
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const size_t vb = (size_t)v * N;
  const int np = block_pairs(N, g, G);
  const uint4 none = make_uint4(0u, 0u, 0u, 0u);
  auto fetch = [&](int i) {
    const int k = pair_of(i, g, G);
    return i < np && k < N ? pairs[vb + k] : none;
  };
  uint4 next = fetch((int)threadIdx.x);
  for (int c = (int)threadIdx.x; c < nc; c += kTlThreads) {
    s_hits[c] = 0ull;
    s_entries[c] = 0u;
  }
  if (threadIdx.x == 0) s_large.n = 0u;
  __syncthreads();
  auto count = [&](int c, uint32_t tiles) {
    atomicAdd(&s_entries[c], 1u);
    // bit b of the tiles to bit 16 b
    const uint32_t lo = (tiles & 1u) | (tiles & 2u) << 15, hi = ((tiles >> 2) & 1u) | (tiles & 8u) << 13;
    atomicAdd((unsigned long long*)&s_hits[c], (unsigned long long)hi << 32 | lo);
  };
  auto count_large = [&](int i, int s0, int ds) {
    const int pair = pair_of(i, g, G);
    for_each_large_cell<false>(pairs[vb + pair], rec + (vb + pair) * 4, cells_x, s0, ds,
                               [&](int c, uint32_t tiles, uint32_t) { count(c, tiles); });
  };
  for (int b = wid * 64; b < np; b += kTlThreads) {
    const uint4 q = next;
    next = fetch(b + lane + kTlThreads);
    uint64_t larges = for_each_cell<false>(
        q, 0u, 0u, cells_x, s_own + wid * 64,
        [&](int c, uint32_t tiles, int, uint32_t, uint32_t, uint32_t) { count(c, tiles); });
    if (larges) larges = keep_large(s_large, larges, b + lane);
    for (; larges; larges &= larges - 1) count_large(b + __ffsll((long long)larges) - 1, 0, 1);
  }
  __syncthreads();
  const int nl = min((int)s_large.n, kLargeMost);
  for (int i = 0; i < nl; ++i)
    count_large(__builtin_amdgcn_readfirstlane((int)s_large.pair[i]), wid, kTlThreads / 64);
  __syncthreads();
  const size_t row = (size_t)cb.matrix[v] + (size_t)g * nc;
  for (int c = (int)threadIdx.x; c < nc; c += kTlThreads) {
    ws.hits[row + c] = s_hits[c];
    ws.entries[row + c] = s_entries[c];
  }
}

__device__ __forceinline__ int view_of_cell(const CellBase& cb, int n_views, int cell) {
  int v = 0;
  for (int k = 1; k < n_views; ++k)
    if (cell >= cb.cell[k]) v = k;
  return v;
}

// Column prefix of the entries, totals of both: 16 cells per block, 64 lanes of it share a
// cell's rows, eight rows' loads in flight together.
constexpr int kTlSegs = 64, kTlCols = 16;
__global__ void __launch_bounds__(kTlSegs * kTlCols)
k_cell_colscan(ViewsArg va, CellBase cb, int n_cells, TlSpace ws) {
  __shared__ uint32_t s_sum[5][kTlSegs][kTlCols];
  const int lane = threadIdx.x % kTlCols, seg = threadIdx.x / kTlCols;
  const int cell = (int)blockIdx.x * kTlCols + lane;
  if (blockIdx.x == 0 && threadIdx.x < kTlCounts) ws.count[threadIdx.x] = 0u;
  const bool ok = cell < n_cells;
  const int v = ok ? view_of_cell(cb, va.n, cell) : 0;
  const ViewDev& V = va.v[v];
  const int nc = view_cells(V), lc = ok ? cell - cb.cell[v] : 0;
  const int G = cb.block[v + 1] - cb.block[v];
  const size_t col = (size_t)cb.matrix[v] + lc;
  const int r0 = seg * G / kTlSegs, r1 = ok ? (seg + 1) * G / kTlSegs : r0;
  uint32_t sum = 0, h[4] = {0u, 0u, 0u, 0u};
  for (int r = r0; r < r1; r += 8) {
    uint32_t x[8];
    uint64_t y[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      x[k] = r + k < r1 ? ws.entries[col + (size_t)(r + k) * nc] : 0u;
      y[k] = r + k < r1 ? ws.hits[col + (size_t)(r + k) * nc] : 0ull;
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      sum += x[k];
#pragma unroll
      for (int b = 0; b < 4; ++b) h[b] += (uint32_t)(y[k] >> (16 * b)) & 0xffffu;
    }
  }
  s_sum[4][seg][lane] = sum;
#pragma unroll
  for (int b = 0; b < 4; ++b) s_sum[b][seg][lane] = h[b];
  __syncthreads();
  if (!ok) return;
  uint32_t run = 0;
  for (int k = 0; k < seg; ++k) run += s_sum[4][k][lane];
  if (seg == kTlSegs - 1) ws.sizes[cell] = run + sum;
  for (int r = r0; r < r1; r += 8) {
    uint32_t x[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) x[k] = r + k < r1 ? ws.entries[col + (size_t)(r + k) * nc] : 0u;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      if (r + k < r1) ws.entries[col + (size_t)(r + k) * nc] = run;
      run += x[k];
    }
  }
  if (seg < 4) {
    const int cx = cells_of(V.tiles_x), tx = 2 * (lc % cx) + (seg & 1), ty = 2 * (lc / cx) + (seg >> 1);
    if (tx < V.tiles_x && ty < V.tiles_y) {
      uint32_t t = 0;
      for (int k = 0; k < kTlSegs; ++k) t += s_sum[seg][k][lane];
      ws.totals[V.tile_base + ty * V.tiles_x + tx] = t;
    }
  }
}

// Inclusive scan over a block of NT lanes, on top of `carry` (which moves past the block).
template <int NT>
__device__ __forceinline__ uint32_t block_scan(uint32_t x, uint32_t* s_warp, uint32_t& carry) {
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const uint32_t incl = (uint32_t)wave_scan((int)x);
  __syncthreads();
  if (lane == 63) s_warp[wid] = incl;
  __syncthreads();
  uint32_t r = carry + incl;
#pragma unroll
  for (int w = 0; w < NT / 64; ++w) {
    const uint32_t s = s_warp[w];
    if (w < wid) r += s;
    carry += s;
  }
  return r;
}

// Exclusive scans of the tiles' hits to ranges (zero for empty tiles) and the instance count,
// and of the cells' entries to their starts; the work items of cells past the small size.
// With more than `cap` instances the render is dropped (empty ranges and cells, overflow[0] |=
// 1); the total is formed in 64 bits, since a wrapped one could fit. overflow[2] keeps the
// largest need that a count holds. Every block sums all tiles for the total and for what
// lies before its own kTlOffPer x 1024 tiles and cells (one block alone took 32 us for the
// 28800 tiles of eight 1280x720 views and 7 for one; now 15 and 6, with the cells' lists).
constexpr int kTlOffThreads = 1024;
constexpr int kTlOffPer = 2;
// This lane's sums of x[0 .. n), and of the first `before` of them.
__device__ __forceinline__ void sum_before(const uint32_t* __restrict__ x, int n, int before, uint64_t& all,
                                           uint32_t& pre) {
  for (int i0 = (int)threadIdx.x; i0 < n; i0 += 8 * kTlOffThreads) {
    uint32_t y[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const int i = i0 + k * kTlOffThreads;
      y[k] = i < n ? x[i] : 0u;
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      all += y[k];
      pre += i0 + k * kTlOffThreads < before ? y[k] : 0u;
    }
  }
}
__global__ void __launch_bounds__(kTlOffThreads)
k_cell_offsets(ViewsArg va, CellBase cb, int32_t n_cells, int64_t cap, uint2* __restrict__ ranges,
               uint32_t* __restrict__ n_inst, uint32_t* __restrict__ overflow, uint32_t* __restrict__ split_counts,
               TlSpace ws) {
  __shared__ uint32_t s_warp[kTlOffThreads / 64];
  __shared__ uint64_t s_sum[2][kTlOffThreads / 64];
  __shared__ uint32_t s_items;
  const int n_tiles = va.total_tiles;
  const int first = (int)blockIdx.x * kTlOffThreads * kTlOffPer;
  const int t0 = first + (int)threadIdx.x * kTlOffPer;
  uint64_t all = 0, call = 0;
  uint32_t pre = 0, cpre = 0;
  uint32_t x[kTlOffPer], c[kTlOffPer], xs = 0, cs = 0;
#pragma unroll
  for (int k = 0; k < kTlOffPer; ++k) {
    x[k] = t0 + k < n_tiles ? ws.totals[t0 + k] : 0u;
    c[k] = t0 + k < n_cells ? ws.sizes[t0 + k] : 0u;
    xs += x[k];
    cs += c[k];
  }
  sum_before(ws.totals, n_tiles, first, all, pre);
  sum_before(ws.sizes, min(n_cells, first), first, call, cpre);
  uint32_t large = 0;  // the lane's cells past the small size
#pragma unroll
  for (int k = 0; k < kTlOffPer; ++k) large += c[k] > (uint32_t)kSortSmall ? 1u : 0u;
  // the sums over the block's lanes, then the lanes' places in the block's own run. (The hits
  // of 2^20 tiles by 2^26 Gaussians leave the block's large cells 16 bits; the sums of earlier
  // tiles and cells fit 32 each where they are used.)
  const uint64_t both = block_sum64<kTlOffThreads>((uint64_t)large << 48 | all, s_sum[0]);
  const uint64_t before = block_sum64<kTlOffThreads>((uint64_t)cpre << 32 | pre, s_sum[1]);
  const uint64_t total = both & ((1ull << 48) - 1ull);
  const uint32_t n_large = (uint32_t)(both >> 48);
  uint32_t at = (uint32_t)before, cell_at = (uint32_t)(before >> 32);
  uint32_t run = block_scan<kTlOffThreads>(xs, s_warp, at) - xs;
  uint32_t crun = block_scan<kTlOffThreads>(cs, s_warp, cell_at) - cs;
  const uint32_t count = instance_word(total);
  const bool dropped = (int64_t)total > cap || count == kTooManyInstances;
  // the places of the cells past the small size among the items, with one atomic per block (one
  // per cell took 6 us more for 2280 of them, and 23 where the cells' sorting blocks did it);
  // before the stores below, which a barrier would wait for
  uint32_t item = 0;
  if (n_large > 0 && !dropped) {
    uint32_t carry = 0;
    item = block_scan<kTlOffThreads>(large, s_warp, carry) - large;
    if (threadIdx.x == 0) s_items = atomicAdd(ws.count + kItems, n_large);
    __syncthreads();
    item += s_items;
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    n_inst[0] = count;
    if ((int64_t)total > cap) atomicOr(overflow, 1u);
    if (count != kTooManyInstances) atomicMax(overflow + 2, count);
  }
  if (blockIdx.x == 0 && threadIdx.x < 2 && split_counts)
    split_counts[threadIdx.x] = 0u;  // (k_cell_sort_small takes the long lists)
#pragma unroll
  for (int k = 0; k < kTlOffPer; ++k) {
    const int i = t0 + k;
    if (i < n_tiles) {
      ranges[i] = x[k] && !dropped ? make_uint2(run, run + x[k]) : make_uint2(0u, 0u);
      const int v = view_of_tile(va, i), lt = i - va.v[v].tile_base, tiles_x = va.v[v].tiles_x;
      const int ty = lt / tiles_x, tx = lt - ty * tiles_x;
      ws.lists[4 * (cb.cell[v] + (ty >> 1) * cells_of(tiles_x) + (tx >> 1)) + 2 * (ty & 1) + (tx & 1)] = run;
    }
    run += x[k];
    if (i >= n_cells) continue;
    if (dropped) crun = c[k] = 0u;
    ws.start[i] = crun;
    if (c[k] > (uint32_t)kSortSmall) ws.items[item++] = make_uint4((uint32_t)i, 0u, crun, c[k]);
    crun += c[k];
    if (i == n_cells - 1) ws.start[n_cells] = crun;
  }
}

// DET: the entry carries, instead of the Gaussian, the emission index of its first hit (the
// pair's first one plus the pair's hits in earlier cells), which grows with the Gaussian, and
// emit_g tells the Gaussian of it.
template <bool DET>
__global__ void __launch_bounds__(kTlThreads) __attribute__((amdgpu_waves_per_eu(8)))
k_cell_place(const float4* __restrict__ rec, const uint4* __restrict__ pairs, const uint32_t* __restrict__ dkey,
             const uint32_t* __restrict__ inst_off, int32_t N, ViewsArg va, CellBase cb, TlSpace ws,
             uint64_t* __restrict__ entries, uint32_t* __restrict__ emit_g) {
  extern __shared__ uint32_t s_pos[];
  __shared__ uint8_t s_own[kTlThreads];
  __shared__ LargeList s_large;
  if (render_dropped(va)) return;
  int g, G;
  const int v = view_of_block(cb, va.n, g, G);
  const ViewDev& V = va.v[v];
  const int nc = view_cells(V), cells_x = cells_of(V.tiles_x);
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const size_t vb = (size_t)v * N;
  const int np = block_pairs(N, g, G);
  uint4 nq;
  uint32_t nd, ne;
  auto fetch = [&](int i) {
    const int k = pair_of(i, g, G);
    nq = make_uint4(0u, 0u, 0u, 0u);
    nd = ne = 0u;
    if (i < np && k < N) {
      nq = pairs[vb + k];
      nd = dkey[vb + k];
      if (DET) ne = inst_off[vb + k];
    }
  };
  fetch((int)threadIdx.x);
  const uint32_t* row = ws.entries + cb.matrix[v] + (size_t)g * nc;
  for (int c = (int)threadIdx.x; c < nc; c += kTlThreads) s_pos[c] = row[c] + ws.start[cb.cell[v] + c];
  if (threadIdx.x == 0) s_large.n = 0u;
  __syncthreads();
  auto place = [&](int c, uint32_t tiles, uint32_t id, uint32_t idx, uint32_t od, uint32_t oe) {
    const uint32_t slot = atomicAdd(&s_pos[c], 1u);
    if (DET) {
      emit_g[oe + idx] = id;
      id = oe + idx;
    }
    entries[slot] = (uint64_t)od << 32 | (id << kTlMaskBits) | tiles;
  };
  auto place_large = [&](int i, int s0, int ds) {
    const int pair = pair_of(i, g, G);
    const uint32_t od = dkey[vb + pair], oe = DET ? inst_off[vb + pair] : 0u;
    for_each_large_cell<DET>(
        pairs[vb + pair], rec + (vb + pair) * 4, cells_x, s0, ds,
        [&](int c, uint32_t tiles, uint32_t idx) { place(c, tiles, (uint32_t)pair, idx, od, oe); });
  };
  for (int b = wid * 64; b < np; b += kTlThreads) {
    const uint4 q = nq;
    const uint32_t d = nd, e0 = ne;
    fetch(b + lane + kTlThreads);
    uint64_t larges = for_each_cell<DET>(q, d, e0, cells_x, s_own + wid * 64,
                                         [&](int c, uint32_t tiles, int own, uint32_t idx, uint32_t od, uint32_t oe) {
                                           place(c, tiles, (uint32_t)pair_of(b + own, g, G), idx, od, oe);
                                         });
    if (larges) larges = keep_large(s_large, larges, b + lane);
    for (; larges; larges &= larges - 1) place_large(b + __ffsll((long long)larges) - 1, 0, 1);
  }
  __syncthreads();
  // (a pair's hits in earlier cells are counted by the wave that walks it: whole pairs then)
  const int nl = min((int)s_large.n, kLargeMost);
  for (int i = DET ? wid : 0; i < nl; i += DET ? kTlThreads / 64 : 1)
    place_large(__builtin_amdgcn_readfirstlane((int)s_large.pair[i]), DET ? 0 : wid, DET ? 1 : kTlThreads / 64);
}

// Orders n <= CAP entries of LDS: a bitonic network in the form whose comparators all point
// the same way, so that entries past n count as larger than all others and are never touched.
template <int NT>
__device__ __forceinline__ void bitonic_sort(uint64_t* s, int n) {
  auto exchange = [&](int i, int j) {
    if (j < n) {
      const uint64_t a = s[i], b = s[j];
      if (b < a) {
        s[i] = b;
        s[j] = a;
      }
    }
  };
  for (int k = 2; (k >> 1) < n; k <<= 1) {
    for (int h = k >> 1; h > 0; h >>= 1) {
      __syncthreads();
      // comparator p: i has bit h clear; its partner mirrors it in the first step of a merge
      for (int p = (int)threadIdx.x;; p += NT) {
        const int i = ((p & ~(h - 1)) << 1) | (p & (h - 1));
        if (i >= n) break;
        exchange(i, h == (k >> 1) ? i ^ (k - 1) : i | h);
      }
    }
  }
  __syncthreads();
}

// One cell (or chunk of one) per block, in LDS. The entries are counted into as many coarse
// bins as lanes, which cut the range of their depth bits evenly; each coarse bin is then cut
// evenly into as many fine bins as half its entries, so that the fine bins follow the depths'
// distribution. Both maps are monotone, so the bins are in order. The entries are scattered
// to their fine bins' places and ranked inside their bin by comparing with its members. (One
// level of 2048 even bins left up to 141 entries in a bin of a street scene's cells, whose
// depths bunch up in front of a far sky: 63 and 85 us for the two sizes where this takes 21
// and 25.) With a bin of more than kBinMost (clusters far narrower than a coarse bin, equal
// depths) a bitonic network orders the entries instead, whose time does not depend on the
// values.
constexpr int kBinMost = 256;
// Up to this many entries are ranked by comparing each with all: two barriers where the bins
// take a dozen (6435 cells of 60 entries on average: 49 us with bins alone, 36 with this; up to
// 512 entries ranked: 40).
constexpr int kRankMost = 128;
// Two fine bins share a word (16 bits each: CAP < 2^16); four 4096-entry blocks fit a CU.
template <int NT, int CAP>
struct __align__(16) SortLds {
  uint64_t e[CAP];
  uint32_t coarse[NT + 1];
  uint32_t bin[CAP / 4 + 1];
  uint32_t warp[NT / 64];
  uint32_t lo, hi, most;
};
__device__ __forceinline__ uint32_t bin_value(const uint32_t* bins, uint32_t b) {
  return (bins[b >> 1] >> (16 * (b & 1u))) & 0xffffu;
}

// Leaves n entries, src(i) for i < n, in order in L.e (after a barrier). (Of more than kRankMost
// all are read before L.e is written.)
template <int NT, int CAP, typename SRC>
__device__ __forceinline__ void sort_run(SortLds<NT, CAP>& L, int n, SRC src) {
  constexpr int PER = CAP / NT, WORDS = CAP / 4 / NT;
  static_assert(CAP % (4 * NT) == 0 && CAP < 65536, "whole words of bins per lane");
  const int tid = (int)threadIdx.x;
  if (CAP <= kSortSmall && n <= kRankMost) {  // (the larger size has none so small)
    const uint64_t e = tid < n ? src(tid) : ~0ull;
    if (tid < kRankMost) L.e[tid] = e;  // (past n: larger than every entry)
    __syncthreads();
    int r = 0;
    if (tid < n)
      for (int j = 0; j < n; j += 8)
#pragma unroll
        for (int u = 0; u < 8; ++u) r += L.e[j + u] < e ? 1 : 0;
    __syncthreads();
    if (tid < n) L.e[r] = e;
    __syncthreads();
    return;
  }
  uint64_t e[PER];
  uint32_t lo = 0xffffffffu, hi = 0u;
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int i = tid + k * NT;
    e[k] = i < n ? src(i) : ~0ull;
    if (i < n) {
      lo = min(lo, (uint32_t)(e[k] >> 32));
      hi = max(hi, (uint32_t)(e[k] >> 32));
    }
  }
  if (tid == 0) {
    L.lo = 0xffffffffu;
    L.hi = 0u;
    L.most = 0u;
  }
  L.coarse[tid] = 0u;
#pragma unroll
  for (int k = 0; k < WORDS; ++k) L.bin[tid + k * NT] = 0u;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    lo = min(lo, (uint32_t)__shfl_xor((int)lo, o, 64));
    hi = max(hi, (uint32_t)__shfl_xor((int)hi, o, 64));
  }
  __syncthreads();
  if ((tid & 63) == 0 && lo <= hi) {
    atomicMin(&L.lo, lo);
    atomicMax(&L.hi, hi);
  }
  __syncthreads();
  lo = L.lo;
  // every step of the map is monotone: difference, conversion, product with a constant, floor
  const float scale = (float)NT / ((float)(L.hi - lo) + 1.0f);
  auto coarse_of = [&](uint64_t x, float& f) {
    f = (float)((uint32_t)(x >> 32) - lo) * scale;
    return min((uint32_t)f, (uint32_t)(NT - 1));
  };
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    if (k * NT >= n) break;  // (uniform)
    float f;
    if (tid + k * NT < n) atomicAdd(&L.coarse[coarse_of(e[k], f)], 1u);
  }
  __syncthreads();
  {
    const uint32_t c = L.coarse[tid];
    uint32_t carry = 0;
    const uint32_t end = block_scan<NT>(c, L.warp, carry);
    L.coarse[tid] = end - c;
    if (tid == 0) L.coarse[NT] = (uint32_t)n;
  }
  __syncthreads();
  uint32_t at[PER];  // fine bin, and the entry's number in it << 16
  uint32_t most = 0;
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    at[k] = 0;
    if (k * NT >= n) break;
    if (tid + k * NT < n) {
      float f;
      const uint32_t b = coarse_of(e[k], f), s = L.coarse[b], c = L.coarse[b + 1] - s;
      const uint32_t fine = (s + min((uint32_t)((f - (float)b) * (float)c), c - 1u)) >> 1;
      const uint32_t sh = 16 * (fine & 1u);
      const uint32_t rank = (atomicAdd(&L.bin[fine >> 1], 1u << sh) >> sh) & 0xffffu;
      at[k] = fine | rank << 16;
      most = max(most, rank + 1u);
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) most = max(most, (uint32_t)__shfl_xor((int)most, o, 64));
  if ((tid & 63) == 0 && most > 0u) atomicMax(&L.most, most);
  __syncthreads();
  if (L.most > (uint32_t)kBinMost) {
#pragma unroll
    for (int k = 0; k < PER; ++k)
      if (tid + k * NT < n) L.e[tid + k * NT] = e[k];
    bitonic_sort<NT>(L.e, n);
    return;
  }
  {
    // exclusive scan of the bins, a run of 2 WORDS per lane
    uint32_t c[WORDS], sum = 0, carry = 0;
    uint32_t* run = L.bin + tid * WORDS;
#pragma unroll
    for (int k = 0; k < WORDS; ++k) {
      c[k] = run[k];
      sum += (c[k] & 0xffffu) + (c[k] >> 16);
    }
    uint32_t start = block_scan<NT>(sum, L.warp, carry) - sum;
#pragma unroll
    for (int k = 0; k < WORDS; ++k) {
      const uint32_t second = start + (c[k] & 0xffffu);
      run[k] = start | second << 16;
      start = second + (c[k] >> 16);
    }
    if (tid == 0) L.bin[CAP / 4] = (uint32_t)n;
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    if (k * NT >= n) break;
    if (tid + k * NT < n) L.e[bin_value(L.bin, at[k] & 0xffffu) + (at[k] >> 16)] = e[k];
  }
  __syncthreads();
  // rank inside the bin, four members' loads in flight together
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    if (k * NT >= n) break;
    if (tid + k * NT < n) {
      const uint32_t b = at[k] & 0xffffu, b0 = bin_value(L.bin, b), b1 = bin_value(L.bin, b + 1);
      uint32_t p = b0;
      for (uint32_t j = b0; j < b1; j += 4) {
        uint64_t x[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) x[u] = L.e[min(j + u, b1 - 1)];
#pragma unroll
        for (int u = 0; u < 4; ++u) p += (j + u < b1 && x[u] < e[k]) ? 1u : 0u;
      }
      at[k] = p;
    }
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    if (k * NT >= n) break;
    if (tid + k * NT < n) L.e[at[k]] = e[k];
  }
  __syncthreads();
}

// Where a cell's tiles' lists go.
struct ListOut {
  uint32_t* list_g;
  uint32_t* list_e;          // nullptr unless deterministic
  const uint32_t* emit_g;
};

// Deals the n ordered entries e of a cell out to its tiles' lists: each wave takes a run of
// 64-entry groups, counts its run's hits per tile, and after a prefix over the waves places
// them, a group at a time, by ballots. to: where the lists start. s_cnt: [waves][4].
template <int NT>
__device__ __forceinline__ void deal_cell(const uint64_t* e, int n, const uint4& to, uint32_t (*s_cnt)[4],
                                          const ListOut& o) {
  constexpr int NW = NT / 64;
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const int groups = (n + 63) >> 6, per = (groups + NW - 1) / NW;
  const int g0 = min(wid * per, groups), g1 = min(g0 + per, groups);
  uint32_t cnt[4] = {0u, 0u, 0u, 0u};
  for (int g = g0; g < g1; ++g) {
    const int i = g * 64 + lane;
    const uint32_t tiles = i < n ? (uint32_t)e[i] & 15u : 0u;
#pragma unroll
    for (int b = 0; b < 4; ++b) cnt[b] += (uint32_t)__popcll(__ballot((tiles >> b) & 1u));
  }
  if (lane < 4) s_cnt[wid][lane] = lane == 0 ? cnt[0] : lane == 1 ? cnt[1] : lane == 2 ? cnt[2] : cnt[3];
  __syncthreads();
  uint32_t at[4] = {to.x, to.y, to.z, to.w};
#pragma unroll
  for (int b = 0; b < 4; ++b)
    for (int w = 0; w < wid; ++w) at[b] += s_cnt[w][b];
  const uint64_t below = lane ? (~0ull >> (64 - lane)) : 0ull;
  for (int g = g0; g < g1; ++g) {
    const int i = g * 64 + lane;
    const uint32_t low = i < n ? (uint32_t)e[i] : 0u;
    const uint32_t tiles = low & 15u, id = low >> kTlMaskBits;
    const uint32_t gid = o.list_e && tiles ? o.emit_g[id] : id;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const uint64_t m = __ballot((tiles >> b) & 1u);
      if ((tiles >> b) & 1u) {
        const uint32_t slot = at[b] + (uint32_t)__popcll(m & below);
        o.list_g[slot] = gid;
        if (o.list_e) o.list_e[slot] = id + (uint32_t)__popc(tiles & ((1u << b) - 1u));
      }
      at[b] += (uint32_t)__popcll(m);
    }
  }
}

// First entry of chunk c where the first `longer` chunks have len + 1 entries and the rest len.
__device__ __forceinline__ int chunk_begin(int len, int longer, int c) { return c * len + min(c, longer); }

// An ordered chunk, back to its place, and per 64 of its entries which of them reach each of
// the cell's four tiles (a 64-bit mask per tile) and how many of the chunk's earlier ones do
// (32 bits each): kGroupWords words per group, the chunk's totals after its last.
constexpr int kGroupWords = 6;
template <int NT>
__device__ __forceinline__ void write_chunk(const uint64_t* e, int n, uint64_t* __restrict__ list,
                                            uint64_t* __restrict__ groups, uint32_t (*s_cnt)[4]) {
  constexpr int NW = NT / 64;
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const int ng = (n + 63) >> 6, per = (ng + NW - 1) / NW;
  const int g0 = min(wid * per, ng), g1 = min(g0 + per, ng);
  uint32_t at[4] = {0u, 0u, 0u, 0u};
  for (int pass = 0; pass < 2; ++pass) {
    for (int g = g0; g < g1; ++g) {
      const int i = g * 64 + lane;
      const uint64_t x = i < n ? e[i] : 0ull;
      if (pass == 0 && i < n) list[i] = x;
      uint64_t m[4];
#pragma unroll
      for (int b = 0; b < 4; ++b) m[b] = __ballot((uint32_t)(x >> b) & 1u);
      if (pass == 1 && lane < kGroupWords)
        groups[g * kGroupWords + lane] = lane == 0   ? m[0]
                                         : lane == 1 ? m[1]
                                         : lane == 2 ? m[2]
                                         : lane == 3 ? m[3]
                                         : lane == 4 ? (uint64_t)at[1] << 32 | at[0]
                                                     : (uint64_t)at[3] << 32 | at[2];
#pragma unroll
      for (int b = 0; b < 4; ++b) at[b] += (uint32_t)__popcll(m[b]);
    }
    if (pass == 0) {
      if (lane < 4) s_cnt[wid][lane] = lane == 0 ? at[0] : lane == 1 ? at[1] : lane == 2 ? at[2] : at[3];
      __syncthreads();
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        at[b] = 0u;
        for (int w = 0; w < wid; ++w) at[b] += s_cnt[w][b];
      }
    } else if (g0 < g1 && g1 == ng && lane < kGroupWords) {
      groups[ng * kGroupWords + lane] = lane < 4 ? 0ull : lane == 4 ? (uint64_t)at[1] << 32 | at[0] : (uint64_t)at[3] << 32 | at[2];
    }
  }
  __syncthreads();  // s_cnt and the entries are reused
}

// Entries first, first + step, ... of chunk c of a cell to its tiles' lists: an entry's place in
// a list is the number of entries before it that reach the tile, in its own chunk and, by a
// binary search, in every other.
__device__ __forceinline__ void merge_chunk(const uint64_t* list, const uint64_t* groups, int n, int nch, int c,
                                            int first, int step, const uint4& to, const ListOut& o) {
  const int len = n / nch, longer = n % nch;
  const int a0 = chunk_begin(len, longer, c), b0 = chunk_begin(len, longer, c + 1);
  for (int i = a0 + first; i < b0; i += step) {
    const uint64_t e = list[i];
    uint32_t at[4] = {to.x, to.y, to.z, to.w};
    for (int k = 0; k < nch; ++k) {
      const int a = chunk_begin(len, longer, k);
      int lo = k == c ? i : a, hi = k == c ? i : chunk_begin(len, longer, k + 1);
      while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (list[mid] < e) lo = mid + 1;
        else hi = mid;
      }
      const uint64_t* g = groups + a + ((lo - a) >> 6) * kGroupWords;
      const uint64_t below = (1ull << ((lo - a) & 63)) - 1ull;
      const uint64_t p0 = g[4], p1 = g[5];
      at[0] += (uint32_t)__popcll(g[0] & below) + (uint32_t)p0;
      at[1] += (uint32_t)__popcll(g[1] & below) + (uint32_t)(p0 >> 32);
      at[2] += (uint32_t)__popcll(g[2] & below) + (uint32_t)p1;
      at[3] += (uint32_t)__popcll(g[3] & below) + (uint32_t)(p1 >> 32);
    }
    const uint32_t tiles = (uint32_t)e & 15u, id = (uint32_t)e >> kTlMaskBits;
    const uint32_t gid = o.list_e ? o.emit_g[id] : id;
#pragma unroll
    for (int b = 0; b < 4; ++b)
      if ((tiles >> b) & 1u) {
        o.list_g[at[b]] = gid;
        if (o.list_e) o.list_e[at[b]] = id + (uint32_t)__popc(tiles & ((1u << b) - 1u));
      }
  }
}

// Orders and deals out cell `cell`, or orders its chunk c where it has several. groups: one word
// per entry, which the chunks' groups fit into.
template <bool LARGE>
__device__ __forceinline__ void sort_cell(SortLds<SortShape<LARGE>::threads, SortShape<LARGE>::cap>& L,
                                          uint32_t (*s_cnt)[4], int cell, int c, uint32_t start, int n,
                                          uint64_t* __restrict__ entries, uint64_t* __restrict__ groups,
                                          const uint32_t* __restrict__ lists, const ListOut& o) {
  constexpr int NT = SortShape<LARGE>::threads;
  uint64_t* list = entries + start;
  const uint4 to = ((const uint4*)lists)[cell];  // (in flight while the entries are ordered)
  const int nch = LARGE ? sort_chunks((uint32_t)n) : 1;
  if (nch == 1) {
    sort_run(L, n, [&](int i) { return list[i]; });
    deal_cell<NT>(L.e, n, to, s_cnt, o);
    return;
  }
  const int len = n / nch, longer = n % nch;
  const int a = chunk_begin(len, longer, c), b = chunk_begin(len, longer, c + 1);
  sort_run(L, b - a, [&](int i) { return list[a + i]; });
  write_chunk<NT>(L.e, b - a, list + a, groups + start + a, s_cnt);
}

// Block c orders cell c's entries where the small size holds them, lists the chunks after the
// first of a cell of several, and marks the cell's long tile lists (split_tile).
__global__ void __launch_bounds__(SortShape<false>::threads)
k_cell_sort_small(ViewsArg va, CellBase cb, const uint2* __restrict__ ranges, uint64_t* __restrict__ entries, TlSpace ws,
                  uint4* __restrict__ extra, ListOut o, SplitArg sp) {
  using S = SortShape<false>;
  __shared__ SortLds<S::threads, S::cap> L;
  __shared__ uint32_t s_cnt[S::threads / 64][4];
  const int cell = (int)blockIdx.x;
  const uint32_t start = ws.start[cell];
  const int n = (int)(ws.start[cell + 1] - start);
  if (n > 0 && n <= S::cap) sort_cell<false>(L, s_cnt, cell, 0, start, n, entries, nullptr, ws.lists, o);
  if (n > kSortMost) {
    const uint32_t more = (uint32_t)sort_chunks((uint32_t)n) - 1u;
    if (threadIdx.x == 0) s_cnt[0][0] = atomicAdd(ws.count + kExtra, more);
    __syncthreads();
    for (uint32_t j = threadIdx.x; j < more; j += S::threads)
      extra[s_cnt[0][0] + j] = make_uint4((uint32_t)cell, j + 1u, start, (uint32_t)n);
  }
  if (sp.par > 0 && threadIdx.x < 4) {
    const int v = view_of_cell(cb, va.n, cell), lc = cell - cb.cell[v];
    const ViewDev& V = va.v[v];
    const int cx = cells_of(V.tiles_x);
    const int tx = 2 * (lc % cx) + ((int)threadIdx.x & 1), ty = 2 * (lc / cx) + ((int)threadIdx.x >> 1);
    if (tx < V.tiles_x && ty < V.tiles_y) {
      const int t = V.tile_base + ty * V.tiles_x + tx;
      const uint2 r = ranges[t];
      split_tile(sp, t, r.y - r.x, *sp.n_inst, va.total_tiles, sp.counts);
    }
  }
}

// Blocks [0, n_items) take one item of the larger cells each (the grid is the most that the
// instances allow: a block per cell spent 15 us on 6435 cells without one such item), the
// others a chunk after a cell's first.
__global__ void __launch_bounds__(SortShape<true>::threads)
k_cell_sort_large(uint64_t* __restrict__ entries, uint64_t* __restrict__ groups, const uint4* __restrict__ items,
                  const uint4* __restrict__ extra, const uint32_t* __restrict__ counts,
                  const uint32_t* __restrict__ lists, int n_items, ListOut o) {
  using S = SortShape<true>;
  __shared__ SortLds<S::threads, S::cap> L;
  __shared__ uint32_t s_cnt[S::threads / 64][4];
  const bool first = (int)blockIdx.x < n_items;
  const uint32_t x = first ? blockIdx.x : blockIdx.x - (uint32_t)n_items;
  const uint4 it = (first ? items : extra)[x];  // (a grid of at most the items' places)
  if (x >= counts[first ? kItems : kExtra]) return;
  sort_cell<true>(L, s_cnt, (int)it.x, (int)it.y, it.z, (int)it.w, entries, groups, lists, o);
}

// Cells of more than kRankChunks chunks are merged in segments of the whole order, three per
// chunk, whose ends are found in all chunks at once: the cost per entry grows with the
// logarithm of the chunks, where an entry's rank takes a search in every other chunk.
constexpr int kRankChunks = 3;
constexpr int kMergeThreads = 1024, kSegMost = 8192, kSegsPerChunk = 3;
// A segment ends within kSegSlack entries of its even share: the largest even share, one such
// distance at either end.
constexpr int kSegSlack = (kSegMost - (kSortMost + kSegsPerChunk - 1) / kSegsPerChunk) / 2;
static_assert(kSortMost * kRankChunks / (kRankChunks + 1) / kSegsPerChunk > 2 * kSegSlack, "ends in order");
constexpr int kMostPlaces = kMergeThreads / 4;  // (more than kRankChunks chunks: four lanes each or more)
static_assert(kRankChunks >= 3, "kMostPlaces");
template <int PER>
union MergeLds {
  static constexpr int chunks = PER * kMergeThreads;
  SortLds<kMergeThreads, kSegMost> sort;
  struct {                           // (where sort.e comes later)
    uint16_t lo[2][chunks], hi[2][chunks];
    uint16_t from[chunks];           // where a chunk's piece of the segment starts in it
    uint16_t at[chunks + 1];         // and in the segment
    uint32_t below[2][kMostPlaces];
    uint32_t places[2];
    uint64_t first, last;
  } find;
  static_assert(sizeof(find) <= sizeof(sort.e), "read while the bins are cleared");
};

// The places in a cell's nch ordered chunks of two values with about r[0] and r[1] of its n
// entries below them: left in F.lo. A round tries kMergeThreads / nch places at once (at least
// one: a lane holds up to PER chunks), each of which counts the entries below it by a binary
// search in every chunk, until a place is within kSegSlack of the rank: what is found depends
// on the cell and the rank alone, so neighbouring segments agree on their common end. The first
// round's places are entries of the first chunk about its own share of the rank (kSpread: two
// standard deviations of it where the chunk is a fair sample); the later ones bisect the range
// of values that is left, and the chunks' own ranges shrink with it. (depth, id) is unique in a
// cell: 64 halvings reach the rank itself.
constexpr int kSpread = 128;
template <int PER, typename FIND>
__device__ __forceinline__ void find_ends(FIND& F, const uint64_t* __restrict__ list, int n, int nch, const int (&r)[2]) {
  constexpr int lanes = 31 - __builtin_clz(kMergeThreads);
  const int tid = (int)threadIdx.x;
  const int lg = min(32 - __builtin_clz(nch - 1), lanes), K = kMergeThreads >> lg;  // places
  const int k = tid >> lg, c0 = tid & ((1 << lg) - 1);                              // place and first chunk
  const int len = n / nch, longer = n % nch;
  if (tid == 0) {
    F.first = ~0ull;
    F.last = 0ull;
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const int c = tid + q * kMergeThreads;
    if (c >= nch) break;
    const int a = chunk_begin(len, longer, c), held = chunk_begin(len, longer, c + 1) - a;
#pragma unroll
    for (int w = 0; w < 2; ++w) {
      F.lo[w][c] = (uint16_t)(r[w] == n ? held : 0);
      F.hi[w][c] = (uint16_t)(r[w] == 0 ? 0 : held);
    }
    atomicMin((unsigned long long*)&F.first, (unsigned long long)list[a]);
    atomicMax((unsigned long long*)&F.last, (unsigned long long)list[a + held - 1]);
  }
  __syncthreads();
  // below L[w] lie less than r[w] entries, below H[w] more
  uint64_t L[2] = {F.first, F.first}, H[2] = {F.last + 1ull, F.last + 1ull};
  bool done[2] = {r[0] == 0 || r[0] == n, r[1] == 0 || r[1] == n};
  for (int round = 0; round < 64 && !(done[0] && done[1]); ++round) {  // (uniform)
    if (tid < 2 * K) F.below[tid >= K][tid & (K - 1)] = 0u;
    if (tid < 2) F.places[tid] = 0u;
    __syncthreads();
    auto place = [&](int w, int i) {
      if (round == 0) {
        const int at = (int)((int64_t)r[w] * len / n) + (2 * i + 1 - K) * kSpread / K;
        return list[min(max(at, 0), len - 1)];
      }
      const uint64_t half = (H[w] - L[w]) >> (lanes - lg + 1);
      return half ? L[w] + (2u * (uint32_t)i + 1u) * half : min(L[w] + (uint64_t)i + 1u, H[w]);
    };
    int lo[PER][2], sum[2] = {0, 0};
    uint64_t v[2] = {0ull, 0ull};
    if (c0 < nch) {
      v[0] = place(0, k);
      v[1] = place(1, k);
    }
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const int c = c0 + q * kMergeThreads;
      lo[q][0] = lo[q][1] = 0;
      if (c >= nch) break;
      const int a = chunk_begin(len, longer, c), held = chunk_begin(len, longer, c + 1) - a;
      int hi[2];
#pragma unroll
      for (int w = 0; w < 2; ++w) {
        lo[q][w] = F.lo[w][c];
        hi[w] = done[w] ? lo[q][w] : F.hi[w][c];
      }
      while (lo[q][0] < hi[0] || lo[q][1] < hi[1]) {
        // (a search that has ended reads the entry at its place, or the last, again)
        const int m0 = (lo[q][0] + hi[0]) >> 1, m1 = (lo[q][1] + hi[1]) >> 1;
        const uint64_t x0 = list[a + min(m0, held - 1)], x1 = list[a + min(m1, held - 1)];
        if (lo[q][0] < hi[0]) {
          if (x0 < v[0]) lo[q][0] = m0 + 1;
          else hi[0] = m0;
        }
        if (lo[q][1] < hi[1]) {
          if (x1 < v[1]) lo[q][1] = m1 + 1;
          else hi[1] = m1;
        }
      }
      sum[0] += lo[q][0];
      sum[1] += lo[q][1];
    }
#pragma unroll
    for (int w = 0; w < 2; ++w)
      if (sum[w] > 0) atomicAdd(&F.below[w][k], (uint32_t)sum[w]);
    __syncthreads();
    if (tid < 2 * K) {
      const int w = tid >= K, i = tid & (K - 1);
      if (F.below[w][i] <= (uint32_t)r[w]) atomicMax(&F.places[w], (uint32_t)i + 1u);
    }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < 2; ++w) {
      if (done[w]) continue;
      const int at = (int)F.places[w];  // places with r entries below or less
      int end = -1;
      if (at > 0 && r[w] - (int)F.below[w][at - 1] <= kSegSlack) end = at - 1;
      else if (at < K && (int)F.below[w][at] - r[w] <= kSegSlack) end = at;
#pragma unroll
      for (int q = 0; q < PER; ++q) {
        const int c = c0 + q * kMergeThreads;
        if (c >= nch) break;
        if (k == (end >= 0 ? end : at - 1)) F.lo[w][c] = (uint16_t)lo[q][w];
        if (k == at) F.hi[w][c] = (uint16_t)lo[q][w];
      }
      done[w] = end >= 0;
      const uint64_t l = at > 0 ? place(w, at - 1) : L[w];
      if (at < K) H[w] = place(w, at);
      L[w] = l;
    }
    __syncthreads();
  }
}

// Segment s of a cell's order to its tiles' lists: its pieces of the chunks are read, ordered
// and dealt out; the lists' places follow from the hits before the pieces.
template <int PER>
__device__ __forceinline__ void merge_segment(MergeLds<PER>& L, uint32_t (*s_cnt)[4], uint32_t* s_warp, uint32_t* s_to,
                                              const uint64_t* __restrict__ list, const uint64_t* __restrict__ groups,
                                              int n, int nch, int s, const uint4& to, const ListOut& o) {
  const int tid = (int)threadIdx.x, lane = tid & 63;
  const int len = n / nch, longer = n % nch, segs = kSegsPerChunk * nch;
  const int r[2] = {(int)((int64_t)s * n / segs), (int)((int64_t)(s + 1) * n / segs)};
  if (tid < 4) s_to[tid] = tid == 0 ? to.x : tid == 1 ? to.y : tid == 2 ? to.z : to.w;
  find_ends<PER>(L.find, list, n, nch, r);
  uint32_t total = 0, hits[4] = {0u, 0u, 0u, 0u};
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    if (q > 0 && q * kMergeThreads >= nch) break;  // (uniform)
    const int c = tid + q * kMergeThreads;
    int p0 = 0, size = 0;
    if (c < nch) {
      p0 = L.find.lo[0][c];
      size = L.find.lo[1][c] - p0;
    }
    const uint32_t end = block_scan<kMergeThreads>((uint32_t)size, s_warp, total);
    if (c >= nch) continue;
    L.find.from[c] = (uint16_t)p0;
    L.find.at[c] = (uint16_t)(end - (uint32_t)size);
    const uint64_t* g = groups + chunk_begin(len, longer, c) + (p0 >> 6) * kGroupWords;
    const uint64_t below = (1ull << (p0 & 63)) - 1ull;
#pragma unroll
    for (int b = 0; b < 4; ++b)
      hits[b] += (uint32_t)__popcll(g[b] & below) + (uint32_t)(g[4 + (b >> 1)] >> (32 * (b & 1)));
  }
  if (tid == 0) L.find.at[nch] = (uint16_t)total;
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    const int x = wave_scan((int)hits[b]);
    if (lane == 63 && x) atomicAdd(&s_to[b], (uint32_t)x);
  }
  __syncthreads();
  const int m = min((int)total, kSegMost);
  sort_run(L.sort, m, [&](int i) {
    int k = 0, past = nch;  // the last piece that starts at or before i (empty ones start where the next does)
    while (past - k > 1) {
      const int mid = (k + past) >> 1;
      if ((int)L.find.at[mid] <= i) k = mid;
      else past = mid;
    }
    return list[chunk_begin(len, longer, k) + L.find.from[k] + (i - L.find.at[k])];
  });
  deal_cell<kMergeThreads>(L.sort.e, m, make_uint4(s_to[0], s_to[1], s_to[2], s_to[3]), s_cnt, o);
  __syncthreads();
}

// Deals out the cells ordered in up to `most` chunks (none in most renders): an entry per lane is
// ranked. The blocks of row y of the grid take the chunks after a cell's first y, y + rows, ...,
// and the first with the second. What bounds it is the chain of an entry's binary searches, 14
// dependent loads per other chunk: 13 us for six cells of some 40000 entries (3 chunks each), 24
// for six of 80000, 23 for one cell of 100k (7), 47 of 200k (13), 67 of 260k (16).
//
// It takes all of a map of up to kRankGaussians (12 chunks: where the worst map, all in one
// cell, costs about as much as merged), and in a crowded image, more than kRankPerCell pairs per
// cell on average, the cells of up to kRankCrowded chunks, which most are there. Elsewhere the
// merge takes the few such cells as well: an idle launch costs 4 us.
constexpr int kRankRows = 32, kRankThreads = 256, kRankCols = kSortMost / kRankThreads;
constexpr int kRankGaussians = 12 * kSortMost;
constexpr int64_t kRankPerCell = 4096;
constexpr int kRankCrowded = 8;
__global__ void __launch_bounds__(kRankThreads)
k_cell_rank(const uint64_t* __restrict__ entries, const uint64_t* __restrict__ groups,
            const uint4* __restrict__ extra, const uint32_t* __restrict__ counts, const uint32_t* __restrict__ lists,
            int most, ListOut o) {
  const uint32_t count = counts[kExtra];
  const bool first = (int)blockIdx.x >= kRankCols;
  const int at = ((int)blockIdx.x % kRankCols) * kRankThreads + (int)threadIdx.x;
  for (uint32_t x = blockIdx.y; x < count; x += kRankRows) {
    const uint4 it = extra[x];
    const int nch = sort_chunks(it.w);
    if (nch > most || (first && it.y != 1u)) continue;
    merge_chunk(entries + it.z, groups + it.z, (int)it.w, nch, first ? 0 : (int)it.y, at, kSortMost,
                ((const uint4*)lists)[it.x], o);
  }
}

// The same for the cells of more than `ranked` chunks, any number of them: the blocks take the
// parts of every chunk after a cell's first in turn, and those of the first where theirs is the
// second. Cells of up to kRankChunks chunks are ranked, the others merged in segments: 34 us for
// one cell of 270k (17 chunks), 88 of 1M (62) and 139 of 2M (123), where ranking took 506 for
// 1M and four times that for 2M. What bounds it is the first round's loads, 64 cold lines per
// wave and step. Its large blocks spread a few chunks worse over the chip than k_cell_rank's: 20
// us for the six cells of 40000, 33 for the six of 80000.
constexpr int kMergeBlocks = 512, kMergeParts = kSortMost / kMergeThreads;
template <int PER>
__global__ void __launch_bounds__(kMergeThreads)
k_cell_merge(const uint64_t* __restrict__ entries, const uint64_t* __restrict__ groups,
             const uint4* __restrict__ extra, const uint32_t* __restrict__ counts, const uint32_t* __restrict__ lists,
             int ranked, ListOut o) {
  __shared__ MergeLds<PER> L;
  __shared__ uint32_t s_cnt[kMergeThreads / 64][4], s_warp[kMergeThreads / 64], s_to[4];
  const uint32_t count = counts[kExtra];
  for (uint32_t u = blockIdx.x; u < 2u * kMergeParts * count; u += kMergeBlocks) {
    const int part = (int)(u / count) % kMergeParts;
    const bool first = u / count >= (uint32_t)kMergeParts;
    const uint4 it = extra[u % count];
    if (first && it.y != 1u) continue;
    const int c = first ? 0 : (int)it.y, n = (int)it.w, nch = sort_chunks(it.w);
    if (nch <= ranked) continue;
    const uint4 to = ((const uint4*)lists)[it.x];
    if (nch <= kRankChunks)
      merge_chunk(entries + it.z, groups + it.z, n, nch, c, part * kMergeThreads + (int)threadIdx.x, kSortMost, to, o);
    else if (part < kSegsPerChunk)
      merge_segment(L, s_cnt, s_warp, s_to, entries + it.z, groups + it.z, n, nch, kSegsPerChunk * c + part, to, o);
  }
}

// tile id of every instance, for inspection
__global__ void __launch_bounds__(256)
k_list_tiles(const uint2* __restrict__ ranges, int64_t cap, uint32_t* __restrict__ tiles) {
  const uint2 r = ranges[blockIdx.x];
  for (int64_t i = (int64_t)r.x + threadIdx.x; i < r.y && i < cap; i += 256) tiles[i] = blockIdx.x;
}

// Dynamic LDS past the 64 KiB that every launch may have is allowed to the kernel by the most
// that any render takes, not by what this one takes: the limit is the kernel's, and renders of
// other maps on other threads set and use it at the same time.
constexpr int kCountLds = 12, kPlaceLds = 4;  // bytes per cell
static_assert(kTlMaxCells * kPlaceLds + 1024 <= 64 * 1024, "k_cell_place needs no allowance");
static hipError_t allow_count_lds(size_t bytes) {
  if (bytes + 1024 <= 64 * 1024) return hipSuccess;
  return hipFuncSetAttribute((const void*)k_cell_count, hipFuncAttributeMaxDynamicSharedMemorySize,
                             kTlMaxCells * kCountLds);
}

hipError_t tile_lists_plan(const float4* rec, const uint4* pairs, int32_t N, const ViewsArg& va, void* space,
                           int64_t cap, uint2* ranges, uint32_t* n_inst, uint32_t* overflow, uint32_t* split_counts,
                           hipStream_t s) {
  const int nc = (int)cells_total(va);
  const CellBase cb = cell_base(va, N);
  const TlSpace ws = tl_space(space, va, cb);
  const dim3 grid((unsigned)cb.block[va.n]);
  const size_t lds = (size_t)max_cells(va) * kCountLds;
  const hipError_t e = allow_count_lds(lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_cell_count, grid, dim3(kTlThreads), lds, s, rec, pairs, N, va, cb,
                     ws);
  hipLaunchKernelGGL(k_cell_colscan, dim3((unsigned)((nc + kTlCols - 1) / kTlCols)), dim3(kTlSegs * kTlCols), 0, s, va, cb,
                     nc, ws);
  const int off_blocks = (va.total_tiles + kTlOffThreads * kTlOffPer - 1) / (kTlOffThreads * kTlOffPer);
  hipLaunchKernelGGL(k_cell_offsets, dim3((unsigned)off_blocks), dim3(kTlOffThreads), 0, s, va, cb, nc, cap,
                     ranges, n_inst, overflow, split_counts, ws);
  return hipGetLastError();
}

hipError_t tile_lists_build(const float4* rec, const uint4* pairs, const uint32_t* dkey, const uint32_t* inst_off,
                            int32_t N, const ViewsArg& va, void* space, const uint2* ranges, uint64_t* entries,
                            uint64_t* groups, void* extra, uint32_t* emit_g, uint32_t* list_g, uint32_t* list_e,
                            const SplitArg& sp, hipStream_t s) {
  const int nc = (int)cells_total(va);
  const CellBase cb = cell_base(va, N);
  const TlSpace ws = tl_space(space, va, cb);
  const dim3 grid((unsigned)cb.block[va.n]);
  const ListOut o{list_g, list_e, emit_g};
  const size_t lds = (size_t)max_cells(va) * kPlaceLds;
  if (list_e)
    hipLaunchKernelGGL(k_cell_place<true>, grid, dim3(kTlThreads), lds, s, rec, pairs, dkey, inst_off, N, va, cb, ws,
                       entries, emit_g);
  else
    hipLaunchKernelGGL(k_cell_place<false>, grid, dim3(kTlThreads), lds, s, rec, pairs, dkey, inst_off, N, va, cb, ws,
                       entries, emit_g);
  hipLaunchKernelGGL(k_cell_sort_small, dim3((unsigned)nc), dim3(SortShape<false>::threads), 0, s, va, cb, ranges,
                     entries, ws, (uint4*)extra, o, sp);
  // a cell holds a Gaussian once: a small map has no items for the larger blocks
  if (N > kSortSmall) {
    const int64_t most = std::min<int64_t>(va.inst_cap, (int64_t)N * nc),
                  items = std::min<int64_t>(nc, most / kSortSmall + 1), more = N > kSortMost ? most_extra(most) : 0;
    hipLaunchKernelGGL(k_cell_sort_large, dim3((unsigned)(items + more)), dim3(SortShape<true>::threads), 0, s, entries,
                       groups, ws.items, (const uint4*)extra, ws.count, ws.lists, (int)items, o);
  }
  const bool crowded = (int64_t)va.n * N > kRankPerCell * nc;
  const int ranked = N <= kRankGaussians ? kMostChunks : crowded ? kRankCrowded : 0;
  if (N > kSortMost && ranked)
    hipLaunchKernelGGL(k_cell_rank, dim3(2 * kRankCols, kRankRows), dim3(kRankThreads), 0, s, entries, groups,
                       (const uint4*)extra, ws.count, ws.lists, ranked, o);
  if (N > kRankGaussians) {
    auto merge = N <= (int64_t)kMergeThreads * kSortMost ? k_cell_merge<1> : k_cell_merge<4>;
    hipLaunchKernelGGL(merge, dim3(kMergeBlocks), dim3(kMergeThreads), 0, s, entries, groups, (const uint4*)extra,
                       ws.count, ws.lists, ranked, o);
  }
  return hipGetLastError();
}

hipError_t list_tiles(const uint2* ranges, int64_t n_tiles, int64_t cap, uint32_t* tiles, hipStream_t s) {
  if (n_tiles <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_list_tiles, dim3((unsigned)n_tiles), dim3(256), 0, s, ranges, cap, tiles);
  return hipGetLastError();
}

}  // namespace gs
