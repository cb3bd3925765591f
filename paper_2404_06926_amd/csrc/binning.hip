// Tile binning by radix sorts (Sec. III-A depth order, Sec. III-D.2 footprint tiles), for the
// images whose cells do not fit the counters of tilelist.hip, and the scans.
//
// The order the blend needs is (global tile, depth, Gaussian index). It is reached in two
// small sorts instead of one wide one:
//   1. a stable LSD radix sort of the (view, Gaussian) pairs by the float bits of their
//      depth (4 passes over V*N 32-bit keys; pairs that reach no tile get the largest key);
//   2. an exclusive scan of the tile counts in that order, then every pair emits its tile
//      ids at its offset, so the instance list comes out in (depth, view-major index)
//      order;
//   3. a stable LSD radix sort of the instances by global tile id only
//      (ceil(log2(tiles + 1)) bits, 2 passes up to 65535 tiles), the values (emission
//      indices) generated by the first pass instead of being written and read;
//   4. [start, end) of every tile in the sorted list.
// Stability makes the result identical to sorting the 64-bit keys tile << 32 | depth bits
// with ties in emission order, at about a fifth of the bytes.
// Kernels that depend on the instance count read it from device memory, so the sequence
// has host-known launch shapes (graph-capturable). A render of more instances than the
// buffers hold drops them all and is flagged; it is then empty.
#include "gs_common.h"
#include "kernels.h"

namespace gs {

constexpr int kScanBlock = 256;
constexpr int kScanItems = 8;   // 2048 elements per block
constexpr int kScanTile = kScanBlock * kScanItems;

// Block-wide exclusive scan of one value per thread; returns the block total.
__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t x, uint32_t* s_warp, uint32_t& total) {
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  uint32_t incl = x;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t y = __shfl_up(incl, o, 64);
    if (lane >= o) incl += y;
  }
  if (lane == 63) s_warp[wid] = incl;
  __syncthreads();
  uint32_t wbase = 0;
  total = 0;
  for (int w = 0; w < (int)(blockDim.x >> 6); ++w) {
    const uint32_t t = s_warp[w];
    if (w < wid) wbase += t;
    total += t;
  }
  __syncthreads();
  return wbase + incl - x;
}

// Exclusive scan over a fixed grid of at most kScanGrid blocks, each owning a contiguous
// run of 2048-element tiles (every block at least one): the up pass sums each block's run,
// the down pass takes the sum of the earlier blocks' runs as its start and scans its tiles
// in order. Element k is in[idx[k]] when idx is given (a gather in another order; the up
// pass stores the gathered values in order so that the down pass reads them contiguously),
// else in[k]; in may equal out.
//
// The scan of the pairs' instance counts also marks, for the emission (below), the pair
// that owns the first instance of every block of kLb instances: pair k owns instances
// [out[k], out[k] + count), and the lane that writes out[k] knows both ends, so it writes
// block_start[b] = k for every b with kLb b in that range (below the capacity). This saves
// the emission a launch of its own for the marks.
constexpr int kScanGrid = 4096;
constexpr int kLbThreads = 256;
constexpr int kLbPer = 2;                      // instances per lane of the emission
constexpr int kLb = kLbThreads * kLbPer;       // instances per emission block

static int scan_grid(int64_t n) {
  return (int)std::min<int64_t>(kScanGrid, std::max<int64_t>(1, (n + kScanTile - 1) / kScanTile));
}

__device__ __forceinline__ void scan_share(int64_t n, int G, int64_t& t0, int64_t& t1) {
  const int64_t nt = (n + kScanTile - 1) / kScanTile;
  t0 = (int64_t)blockIdx.x * nt / G;
  t1 = (int64_t)(blockIdx.x + 1) * nt / G;
}

// GATHER: element k is in[idx[k]], stored in order to gathered[k] as well. A lane's
// indices are loaded first, then all its gathers, then the stores, so that each group of
// loads is in flight together (one round trip each instead of one per element). Loads past
// the end read the last element (clamped, so they need no branch) and count as zero.
template <bool GATHER>
__global__ void __launch_bounds__(kScanBlock)
k_scan_up(const uint32_t* __restrict__ in, const uint32_t* __restrict__ idx, int64_t n, uint64_t* __restrict__ sums,
          int G, uint32_t* __restrict__ gathered) {
  __shared__ uint64_t s_sum[kScanBlock / 64];
  int64_t t0, t1;
  scan_share(n, G, t0, t1);
  uint64_t tsum = 0;
  for (int64_t t = t0; t < t1; ++t) {
    const int64_t base = t * kScanTile + (int64_t)threadIdx.x;
    uint32_t ix[kScanItems], v[kScanItems];
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
      const int64_t e = min(base + (int64_t)k * kScanBlock, n - 1);  // coalesced over the lanes
      ix[k] = GATHER ? idx[e] : (uint32_t)e;
    }
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
      const int64_t e = base + (int64_t)k * kScanBlock;
      const uint32_t x = in[GATHER ? (int64_t)ix[k] : min(e, n - 1)];
      v[k] = e < n ? x : 0u;
    }
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
      const int64_t e = base + (int64_t)k * kScanBlock;
      if (GATHER && e < n) gathered[e] = v[k];
      tsum += v[k];
    }
  }
  tsum = block_sum64<kScanBlock>(tsum, s_sum);
  if (threadIdx.x == 0) sums[blockIdx.x] = tsum;
}

// total (optional): the sum of all elements as an instance count (instance_word), written by
// the last block; the scan itself is modulo 2^32. block_start
// (optional): the emission blocks' first pairs, for instances below bs_cap.
__global__ void __launch_bounds__(kScanBlock)
k_scan_down(const uint32_t* __restrict__ in, const uint32_t* __restrict__ idx, uint32_t* __restrict__ out, int64_t n,
            const uint64_t* __restrict__ sums, int G, uint32_t* __restrict__ total_out,
            uint32_t* __restrict__ block_start, int64_t bs_cap) {
  __shared__ uint32_t s_warp[kScanBlock / 64];
  __shared__ uint64_t s_sum[kScanBlock / 64];
  // start of this block's run: the sums of the blocks before it (G <= 4096: 16 per thread)
  uint64_t before = 0;
#pragma unroll
  for (int k = 0; k < kScanGrid / kScanBlock; ++k) {
    const int b = (int)threadIdx.x + k * kScanBlock;
    if (b < (int)blockIdx.x) before += sums[b];
  }
  before = block_sum64<kScanBlock>(before, s_sum);
  uint32_t carry = (uint32_t)before;
  int64_t t0, t1;
  scan_share(n, G, t0, t1);
  for (int64_t t = t0; t < t1; ++t) {
    const int64_t base = t * kScanTile + (int64_t)threadIdx.x * kScanItems;
    const bool full = base + kScanItems <= n;  // the lane's 8 elements as two 16-B accesses
    uint32_t v[kScanItems];
    uint32_t tsum = 0;
    if (full && !idx) {
      const uint4 a = *(const uint4*)(in + base), b = *(const uint4*)(in + base + 4);
      v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w; v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
    } else {
#pragma unroll
      for (int k = 0; k < kScanItems; ++k) {
        v[k] = 0u;
        if (base + k < n) v[k] = idx ? in[idx[base + k]] : in[base + k];
      }
    }
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) tsum += v[k];
    uint32_t tile_total;
    uint32_t run = carry + block_exclusive_scan(tsum, s_warp, tile_total);
    uint32_t o[kScanItems];
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
      o[k] = run;
      run += v[k];
    }
    if (full) {
      *(uint4*)(out + base) = make_uint4(o[0], o[1], o[2], o[3]);
      *(uint4*)(out + base + 4) = make_uint4(o[4], o[5], o[6], o[7]);
    } else {
#pragma unroll
      for (int k = 0; k < kScanItems; ++k)
        if (base + k < n) out[base + k] = o[k];
    }
    if (block_start) {
#pragma unroll
      for (int k = 0; k < kScanItems; ++k) {
        const int64_t e = min((int64_t)o[k] + v[k], bs_cap);  // v[k] = 0 past n
        for (int64_t b = ((int64_t)o[k] + kLb - 1) / kLb; b * kLb < e; ++b) block_start[b] = (uint32_t)(base + k);
      }
    }
    carry += tile_total;
  }
  if (total_out && blockIdx.x == (unsigned)(G - 1) && threadIdx.x == 0)
    total_out[0] = instance_word(before + sums[G - 1]);
}

// block sums (8 B each), then room for n gathered values
int64_t scan_temp_elems(int64_t n) { return 2 * kScanGrid + n + 1; }

static hipError_t scan_impl(const uint32_t* in, const uint32_t* idx, uint32_t* out, int64_t n, uint32_t* temp,
                            uint32_t* total, uint32_t* block_start, int64_t bs_cap, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const int G = scan_grid(n);
  uint64_t* sums = (uint64_t*)temp;
  uint32_t* gathered = temp + 2 * kScanGrid;
  if (idx)
    hipLaunchKernelGGL(k_scan_up<true>, dim3(G), dim3(kScanBlock), 0, s, in, idx, n, sums, G, gathered);
  else
    hipLaunchKernelGGL(k_scan_up<false>, dim3(G), dim3(kScanBlock), 0, s, in, idx, n, sums, G, gathered);
  hipLaunchKernelGGL(k_scan_down, dim3(G), dim3(kScanBlock), 0, s, idx ? gathered : in, nullptr, out, n, sums, G, total,
                     bs_cap > 0 ? block_start : nullptr, bs_cap);
  return hipGetLastError();
}

// Exclusive scan of n u32 values (in may equal out); temp holds scan_temp_elems(n).
hipError_t exclusive_scan(const uint32_t* in, uint32_t* out, int64_t n, uint32_t* temp, hipStream_t s) {
  return scan_impl(in, nullptr, out, n, temp, nullptr, nullptr, 0, s);
}

hipError_t scan_counts(const uint32_t* counts, const uint32_t* order, uint32_t* offsets, int64_t n,
                       uint32_t* temp, uint32_t* total, uint32_t* block_start, int64_t capacity, hipStream_t s) {
  return scan_impl(counts, order, offsets, n, temp, total, block_start, capacity, s);
}

// ------------------------------------------------------------------ radix sort
// Stable LSD sort with 8-bit digits over a fixed grid of G blocks (even share: block g
// owns a contiguous run of 2048-key tiles, whatever the key count). Each pass:
//   up:      per-block digit counts (digit-major, counts[d * G + g]), one LDS atomic
//            per key into a per-wave histogram;
//   rowscan: one block per digit scans its row over the G blocks and writes the digit
//            total;
//   down:    each block takes the exclusive scan of the 256 digit totals plus its row
//            prefix as the global start of each digit, then walks its tiles in order:
//            every wave ranks its keys with ballot-based peer masks, the tile is placed
//            in LDS in (digit, original order) order and written out by consecutive lanes
//            (each digit's run goes to consecutive addresses), and the digit starts
//            advance by the tile's counts.
// Three launches per pass and a count matrix of 256 x G entries, independent of n.
constexpr int kSortBlock = 256;
constexpr int kSortItems = 8;
constexpr int kSortTile = kSortBlock * kSortItems;  // 2048 keys per tile
constexpr int kWaves = kSortBlock / 64;
constexpr int kSortGrid = 1024;                     // blocks of the up and down sweeps

// Elements to process: all of them when they fit, none after an overflow (the render is
// then empty and the overflow flag tells the host to re-plan).
__device__ __forceinline__ uint32_t sort_count(const uint32_t* n_dev, int64_t cap) {
  const uint32_t n = n_dev[0];
  return (int64_t)n <= cap ? n : 0u;
}

// Tiles [t0, t1) of logical block g among G for n keys.
__device__ __forceinline__ void sort_share(uint32_t n, int G, int g, int64_t& t0, int64_t& t1) {
  const int64_t nt = ((int64_t)n + kSortTile - 1) / kSortTile;
  t0 = (int64_t)g * nt / G;
  t1 = (int64_t)(g + 1) * nt / G;
}

// Lanes of the wave whose digit equals this lane's (one ballot per digit bit: eight, or with
// NARROW only the digit's `bits` < 8), restricted to `ok` lanes.
template <bool NARROW>
__device__ __forceinline__ uint64_t digit_peers(uint32_t d, bool ok, int bits) {
  uint64_t peers = __ballot(ok);
#pragma unroll
  for (int b = 0; b < 8; ++b) {
    if (NARROW && b >= bits) break;  // wave-uniform
    const uint64_t m = __ballot((d >> b) & 1u);
    peers &= ((d >> b) & 1u) ? m : ~m;
  }
  return peers;
}

template <typename K>
__global__ void __launch_bounds__(kSortBlock)
k_radix_up(const K* __restrict__ keys, const uint32_t* __restrict__ n_dev, int64_t cap, int shift,
           uint32_t mask, uint32_t* __restrict__ counts, int G) {
  __shared__ uint32_t s_h[kWaves][256];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  for (int d = lane; d < 256; d += 64) s_h[wid][d] = 0;
  __syncthreads();
  const uint32_t n = sort_count(n_dev, cap);
  const int g = xcd_block((int)blockIdx.x, G);
  int64_t t0, t1;
  sort_share(n, G, g, t0, t1);
  // the next tile's keys are loaded while this one is counted
  K nk[kSortItems];
  auto fetch = [&](int64_t t) {
    const int64_t b = t * kSortTile + (int64_t)wid * (64 * kSortItems);
#pragma unroll
    for (int r = 0; r < kSortItems; ++r) {
      const int64_t idx = b + r * 64 + lane;
      nk[r] = idx < n ? keys[idx] : (K)0;
    }
  };
  if (t0 < t1) fetch(t0);
  for (int64_t t = t0; t < t1; ++t) {
    const int64_t base = t * kSortTile + (int64_t)wid * (64 * kSortItems);
    K k[kSortItems];
#pragma unroll
    for (int r = 0; r < kSortItems; ++r) k[r] = nk[r];
    if (t + 1 < t1) fetch(t + 1);
#pragma unroll
    for (int r = 0; r < kSortItems; ++r) {
      const int64_t idx = base + r * 64 + lane;
      // one LDS atomic per key: the LDS unit serialises the lanes of equal digits, which
      // costs less than the ballots that would rank them (counting needs no order)
      if (idx < n) atomicAdd(&s_h[wid][(uint32_t)(k[r] >> shift) & mask], 1u);
    }
  }
  __syncthreads();
  const int d = threadIdx.x;
  counts[(int64_t)d * G + g] = s_h[0][d] + s_h[1][d] + s_h[2][d] + s_h[3][d];
}

// Block d: exclusive scan of row d (G <= kSortGrid entries) in place, its total to totals[d].
__global__ void __launch_bounds__(256)
k_radix_rowscan(uint32_t* __restrict__ counts, int G, uint32_t* __restrict__ totals) {
  constexpr int kPer = kSortGrid / 256;
  __shared__ uint32_t s_warp[4];
  uint32_t* row = counts + (int64_t)blockIdx.x * G;
  uint32_t v[kPer], sum = 0;
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int i = (int)threadIdx.x * kPer + k;
    v[k] = i < G ? row[i] : 0u;
    sum += v[k];
  }
  uint32_t total;
  uint32_t run = block_exclusive_scan(sum, s_warp, total);
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int i = (int)threadIdx.x * kPer + k;
    if (i < G) row[i] = run;
    run += v[k];
  }
  if (threadIdx.x == 0) totals[blockIdx.x] = total;
}

template <typename K, bool NARROW>
__global__ void __launch_bounds__(kSortBlock)
k_radix_down(const K* __restrict__ kin, const uint32_t* __restrict__ vin, K* __restrict__ kout,
             uint32_t* __restrict__ vout, const uint32_t* __restrict__ n_dev, int64_t cap, int shift, uint32_t mask,
             const uint32_t* __restrict__ counts, const uint32_t* __restrict__ totals, int G) {
  __shared__ uint32_t s_cnt[kWaves][256];   // keys per (wave, digit), then the wave's offset
  __shared__ uint32_t s_start[256];         // first LDS slot of each digit in the tile
  __shared__ uint32_t s_tot[256];           // keys of each digit in the tile
  __shared__ uint32_t s_base[256];          // global position of the block's next key of each digit
  __shared__ uint32_t s_warp[kWaves];
  __shared__ K s_key[kSortTile];
  __shared__ uint32_t s_val[kSortTile];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const uint32_t n = sort_count(n_dev, cap);
  const int g = xcd_block((int)blockIdx.x, G);
  int64_t t0, t1;
  sort_share(n, G, g, t0, t1);
  if (t0 >= t1) return;
  {
    const int d = threadIdx.x;
    uint32_t all;
    const uint32_t start = block_exclusive_scan(totals[d], s_warp, all);
    s_base[d] = start + counts[(int64_t)d * G + g];
  }
  const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  // the next tile's keys and values are loaded into registers while this one is ranked,
  // placed and written
  K nkey[kSortItems];
  uint32_t nval[kSortItems];
  auto fetch = [&](int64_t t) {
    const int64_t b = t * kSortTile + (int64_t)wid * (64 * kSortItems);
#pragma unroll
    for (int r = 0; r < kSortItems; ++r) {
      const int64_t idx = b + r * 64 + lane;
      const bool ok = idx < n;
      nkey[r] = ok ? kin[idx] : (K)0;
      nval[r] = ok ? (vin ? vin[idx] : (uint32_t)idx) : 0u;  // no vin: the values are the positions
    }
  };
  fetch(t0);
  for (int64_t t = t0; t < t1; ++t) {
    for (int d = lane; d < 256; d += 64) s_cnt[wid][d] = 0;
    const int64_t blk0 = t * kSortTile;
    const int64_t base = blk0 + (int64_t)wid * (64 * kSortItems);
    K key[kSortItems];
    uint32_t val[kSortItems], rank[kSortItems], dig[kSortItems];
#pragma unroll
    for (int r = 0; r < kSortItems; ++r) {
      key[r] = nkey[r];
      val[r] = nval[r];
    }
    if (t + 1 < t1) fetch(t + 1);
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kSortItems; ++r) {
      const int64_t idx = base + r * 64 + lane;
      const bool ok = idx < n;
      const uint32_t d = (uint32_t)(key[r] >> shift) & mask;
      dig[r] = d;
      const uint64_t peers = digit_peers<NARROW>(d, ok, __popc(mask));
      uint32_t prev = 0;
      const int leader = peers ? (__ffsll((long long)peers) - 1) : 0;
      if (ok && lane == leader) {
        prev = s_cnt[wid][d];
        s_cnt[wid][d] = prev + (uint32_t)__popcll(peers);
      }
      prev = __shfl(prev, leader, 64);
      rank[r] = prev + (uint32_t)__popcll(peers & lt);
    }
    __syncthreads();
    // digit totals of the tile, their exclusive scan (LDS start of each digit) and each
    // wave's offset inside its digit run
    {
      const int d = threadIdx.x;
      uint32_t tot = 0;
#pragma unroll
      for (int w = 0; w < kWaves; ++w) {
        const uint32_t c = s_cnt[w][d];
        s_cnt[w][d] = tot;
        tot += c;
      }
      uint32_t all;
      s_start[d] = block_exclusive_scan(tot, s_warp, all);
      s_tot[d] = tot;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kSortItems; ++r) {
      const int64_t idx = base + r * 64 + lane;
      if (idx < n) {
        const uint32_t slot = s_start[dig[r]] + s_cnt[wid][dig[r]] + rank[r];
        s_key[slot] = key[r];
        s_val[slot] = val[r];
      }
    }
    __syncthreads();
    const int64_t nblk = min((int64_t)kSortTile, (int64_t)n - blk0);
    for (int i = threadIdx.x; i < nblk; i += kSortBlock) {
      const K k = s_key[i];
      const uint32_t d = (uint32_t)(k >> shift) & mask;
      const uint32_t pos = s_base[d] + ((uint32_t)i - s_start[d]);
      kout[pos] = k;
      vout[pos] = s_val[i];
    }
    __syncthreads();
    s_base[threadIdx.x] += s_tot[threadIdx.x];
  }
}

static int sort_grid(int64_t cap) {
  return (int)std::min<int64_t>(kSortGrid, std::max<int64_t>(1, (cap + kSortTile - 1) / kSortTile));
}

int64_t sort_temp_elems(int64_t cap) { return 256 * (int64_t)sort_grid(cap) + 256; }

// Sorts (keys[0], vals[0]) on bits [0, nbits) using (keys[1], vals[1]) as the double buffer;
// *which receives the index of the buffer that holds the result. vals_iota: vals[0] is not
// read, the values are taken to be 0, 1, 2, ... (the first pass generates them).
hipError_t radix_sort_u32(uint32_t* keys[2], uint32_t* vals[2], const uint32_t* n_dev, int64_t cap, int nbits,
                          uint32_t* temp, int* which, hipStream_t s, bool vals_iota) {
  *which = 0;
  if (cap <= 0) return hipSuccess;
  const int G = sort_grid(cap);
  uint32_t* counts = temp;
  uint32_t* totals = temp + (int64_t)256 * G;
  // as many passes as 8-bit digits need, the bits spread evenly over them: fewer digit
  // values per pass give longer runs of equal digits in each tile, so the scatter writes
  // longer contiguous pieces (12-bit tile ids: two 6-bit passes rather than 8 + 4)
  const int passes = (nbits + 7) / 8;
  const int width = passes ? (nbits + passes - 1) / passes : 8;
  int cur = 0;
  for (int shift = 0; shift < nbits; shift += width) {
    const int w = std::min(width, nbits - shift);
    const uint32_t mask = (w >= 32) ? 0xFFFFFFFFu : ((1u << w) - 1u);
    hipLaunchKernelGGL(k_radix_up<uint32_t>, dim3(G), dim3(kSortBlock), 0, s, keys[cur], n_dev, cap, shift, mask,
                       counts, G);
    hipLaunchKernelGGL(k_radix_rowscan, dim3(256), dim3(256), 0, s, counts, G, totals);
    const uint32_t* vin = (vals_iota && shift == 0) ? nullptr : vals[cur];
    // digits narrower than 8 bits (the tile sort's) skip the ranking ballots of the bits
    // they lack
    if (w < 8)
      hipLaunchKernelGGL((k_radix_down<uint32_t, true>), dim3(G), dim3(kSortBlock), 0, s, keys[cur], vin,
                         keys[cur ^ 1], vals[cur ^ 1], n_dev, cap, shift, mask, counts, totals, G);
    else
      hipLaunchKernelGGL((k_radix_down<uint32_t, false>), dim3(G), dim3(kSortBlock), 0, s, keys[cur], vin,
                         keys[cur ^ 1], vals[cur ^ 1], n_dev, cap, shift, mask, counts, totals, G);
    cur ^= 1;
  }
  *which = cur;
  return hipGetLastError();
}

// Instances are emitted in depth order: pair k of the depth order ((view, Gaussian) id
// order[k]) owns the instance range [offsets[k], offsets[k] + count). Two instances per
// lane, so the work does not depend on how unevenly the counts fall and each block's two
// dependent global round trips (stage the pairs, then gather their records) are shared by
// 512 instances: block b covers instances [512 b, 512 b + 512); it stages the offsets and
// ids of the (at most 512) pairs from block_start[b] in LDS, each pair marking the slot
// where its instances start; an instance's pair is the last mark at or before it (a ballot
// of the marks per 64-slot group), and
// its tile comes from the pair's 64-bit hit mask (its r-th set bit, row-major in the pair's tile
// rectangle). A pair whose rectangle has more than 64 tiles (no mask) is emitted whole by
// the block where its instances start: after the block's own slots, one wave per such pair
// evaluates the tile predicate over the rectangle and places the hits with a ballot prefix
// sum (the blocks its instances reach further on skip them). With more instances
// than the capacity none is written; the overflow flag is raised and the render is emptied
// downstream.
constexpr int kLbGroups = kLb / 64;            // 64-slot mark groups per block

// block_start[b] = the pair that owns instance kLb b (as the scan of the counts marks them).
__global__ void __launch_bounds__(256)
k_block_starts(const uint32_t* __restrict__ offsets, const uint32_t* __restrict__ n_dev, int64_t n_pairs,
               int64_t capacity, uint32_t* __restrict__ block_start) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n_pairs) return;
  const int64_t total = n_dev[0];
  const int64_t o = offsets[k];
  const int64_t e = min(k + 1 < n_pairs ? (int64_t)offsets[k + 1] : total, min(total, capacity));
  for (int64_t b = (o + kLb - 1) / kLb; b * kLb < e; ++b) block_start[b] = (uint32_t)k;
}

__global__ void __launch_bounds__(kLbThreads)
k_dup_lb(const float4* __restrict__ rec, const uint32_t* __restrict__ order, const uint32_t* __restrict__ offsets,
         const uint32_t* __restrict__ counts, const uint32_t* __restrict__ block_start,
         const uint32_t* __restrict__ n_dev, int64_t n_pairs, int32_t N, ViewsArg va, int64_t capacity,
         uint32_t* __restrict__ tiles_out, uint32_t* __restrict__ emit_g, uint32_t* __restrict__ inst_off,
         int all_off, uint32_t* __restrict__ overflow) {
  __shared__ uint32_t s_off[kLb];
  __shared__ uint32_t s_vi[kLb];
  __shared__ uint4 s_r3[kLb];    // tile rectangle and hit mask of the staged pairs that own slots here
  __shared__ int s_mark[kLb];    // staged pair whose instances start at this slot, or -1
  __shared__ int s_glast[kLbGroups];
  __shared__ int s_big[kLb];     // staged pairs that start here and have more than 64 candidate tiles
  __shared__ int s_nbig;
  const int64_t total = n_dev[0];
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    if (total > capacity) atomicOr(overflow, 1u);
    // the largest need since the last check
    if (total != (int64_t)kTooManyInstances) atomicMax(overflow + 2, (uint32_t)total);
  }
  // a dropped render emits nothing (past 2^32 instances the offsets and marks wrapped around)
  const int64_t lim = total > capacity ? 0 : total;
  const int64_t slot0 = (int64_t)blockIdx.x * kLb;
  if (slot0 >= lim) return;
  const int64_t k0 = block_start[blockIdx.x];
  // the pairs that own slots of this block end at the one that holds the next block's
  // first slot (the last block stages up to kLb pairs)
  const int64_t k_last = slot0 + kLb < lim ? (int64_t)block_start[blockIdx.x + 1] : k0 + kLb - 1;
  const int np = (int)min((int64_t)kLb, k_last - k0 + 1);
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
#pragma unroll
  for (int u = 0; u < kLbPer; ++u) s_mark[u * kLbThreads + threadIdx.x] = -1;
  if (threadIdx.x == 0) s_nbig = 0;
  __syncthreads();
  // the pairs k0 .. k0 + np - 1 cover this block (every pair before the unused ones has a
  // tile); a pair marks the slot where its instances start, the last of several pairs
  // with the same offset (the earlier ones have no instance) winning
#pragma unroll
  for (int u = 0; u < kLbPer; ++u) {
    const int p = u * kLbThreads + (int)threadIdx.x;
    if (p >= np) continue;
    const int64_t k = k0 + p;
    const uint32_t vi = k < n_pairs ? order[k] : 0u;
    s_vi[p] = vi;
    const int64_t o = k < n_pairs ? (int64_t)offsets[k] : total;
    s_off[p] = (uint32_t)o;
    if (o >= slot0 && o < slot0 + kLb) atomicMax(&s_mark[o - slot0], p);
    // one record read per pair that owns slots of this block (the first pair and those
    // that start inside it), not one per instance
    const bool starts = o >= slot0 && o < slot0 + kLb;
    if (k < n_pairs && (p == 0 || starts)) {
      const uint4 r3 = *(const uint4*)(rec + (size_t)vi * 4 + 3);
      s_r3[p] = r3;
      const int rw = (int)(r3.y & 0xffff) - (int)(r3.x & 0xffff) + 1, rh = (int)(r3.y >> 16) - (int)(r3.x >> 16) + 1;
      // (a pair without instances starts where the next one does, and the projection wrote
      // no record for it: only pairs with instances are taken)
      if (starts && rw * rh > 64 && counts[vi] > 0u) s_big[atomicAdd(&s_nbig, 1)] = p;
    }
  }
  __syncthreads();
  // owner of each slot: the last mark at or before it (slot0 itself belongs to staged pair
  // 0 by the choice of k0); within a 64-slot group from a ballot of the marks, across
  // groups from the last mark of each earlier group. Slot u kLbThreads + t lies in group
  // u (kLbThreads / 64) + wave.
  uint64_t marks[kLbPer];
#pragma unroll
  for (int u = 0; u < kLbPer; ++u) {
    const int g = u * (kLbThreads / 64) + wid;
    marks[u] = __ballot(s_mark[u * kLbThreads + threadIdx.x] >= 0);
    if (lane == 0) s_glast[g] = marks[u] ? s_mark[g * 64 + 63 - __clzll((long long)marks[u])] : -1;
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < kLbPer; ++u) {
    const int g = u * (kLbThreads / 64) + wid;
    const int64_t slot = slot0 + u * kLbThreads + threadIdx.x;
    if (slot >= lim) continue;
    const uint64_t upto = marks[u] & (~0ull >> (63 - lane));
    int lo = 0;
    if (upto) {
      lo = s_mark[g * 64 + 63 - __clzll((long long)upto)];
    } else {
      for (int gg = 0; gg < g; ++gg) lo = max(lo, s_glast[gg]);
    }
    const uint32_t vi = s_vi[lo];
    const uint32_t r = (uint32_t)(slot - (int64_t)s_off[lo]);
    const uint4 r3 = s_r3[lo];
    const uint32_t a = r3.x, b = r3.y;
    const int x0 = a & 0xffff, y0 = a >> 16, x1 = b & 0xffff, y1 = b >> 16;
    const int rw = x1 - x0 + 1;
    const bool big = rw * (y1 - y0 + 1) > 64;
    // the first emission index of every pair, for the deterministic backward (all_off)
    if (r == 0 && all_off) inst_off[vi] = (uint32_t)slot;
    if (big) continue;  // written by the block where the pair starts (below)
    const uint32_t mlo = r3.z, mhi = r3.w;
    const uint32_t clo = (uint32_t)__popc(mlo);
    const int pos = r < clo ? nth_set_bit32(mlo, r) : 32 + nth_set_bit32(mhi, r - clo);
    // pair index -> (view, Gaussian); one view needs no division
    const int v = va.n == 1 ? 0 : (int)(vi / (uint32_t)N);
    const uint32_t gid = vi - (uint32_t)v * (uint32_t)N;
    const ViewDev& V = va.v[v];
    // row and column of the hit in the rectangle: pos < 64 and rw <= 64, so the quotient's
    // fractional part is a multiple of 1 / rw >= 1 / 64 and pos / rw is within 64 x 2^-23 of
    // pos * rcp(rw): adding 1 / 128 before truncating gives the exact quotient
    const int qy = (int)fmaf((float)pos, __builtin_amdgcn_rcpf((float)rw), 1.0f / 128.0f);
    const int qx = pos - qy * rw;
    tiles_out[slot] = (uint32_t)(V.tile_base + (y0 + qy) * V.tiles_x + (x0 + qx));
    emit_g[slot] = gid;
  }
  // the pairs with more than 64 candidate tiles that start in this block, one wave each
  const int nbig = s_nbig;
  const uint64_t below = lane ? (~0ull >> (64 - lane)) : 0ull;  // lanes under this one
  for (int q = wid; q < nbig; q += kLbThreads / 64) {
    const int sp = s_big[q];
    const uint32_t vi = s_vi[sp];
    const int64_t o = s_off[sp];
    const int v = va.n == 1 ? 0 : (int)(vi / (uint32_t)N);
    const uint32_t g = vi - (uint32_t)v * (uint32_t)N;
    const ViewDev& V = va.v[v];
    const float4* rp = rec + (size_t)vi * 4;
    const float4 r0 = rp[0], r1 = rp[1], r2 = rp[2];
    const uint32_t a = s_r3[sp].x, b = s_r3[sp].y;
    const int x0 = a & 0xffff, y0 = a >> 16, x1 = b & 0xffff, y1 = b >> 16;
    const int rw = x1 - x0 + 1, area = rw * (y1 - y0 + 1);
    const uint32_t cnt = counts[vi];
    uint32_t base = 0;
    // (wave-uniform bound: the walk ends at the rectangle's end or the pair's last hit)
    for (int t0 = 0; t0 < area && base < cnt; t0 += 64) {
      const int t = t0 + lane;
      int tx = 0, ty = 0;
      bool hit = false;
      if (t < area) {
        tx = x0 + t % rw;
        ty = y0 + t / rw;
        hit = key_tile_hit(r0.x, r0.y, r0.z, r0.w, r1.x, r2.w, tx, ty);
      }
      const uint64_t m = __ballot(hit);
      const uint32_t p = base + (uint32_t)__popcll(m & below);
      if (hit && p < cnt) {
        const int64_t slot = o + p;
        tiles_out[slot] = (uint32_t)(V.tile_base + ty * V.tiles_x + tx);
        emit_g[slot] = g;
      }
      base += (uint32_t)__popcll(m);
    }
    // unreachable when both passes agree; the sentinel tile sorts after every real tile
    for (uint32_t p = base + lane; p < cnt; p += 64) {
      tiles_out[o + p] = 0xffffffffu;
      emit_g[o + p] = 0u;
    }
  }
}

int64_t block_start_elems(int64_t capacity) { return capacity / kLb + 2; }

hipError_t duplicate_keys(const float4* rec, const uint32_t* counts, const uint32_t* order, const uint32_t* offsets,
                          const uint32_t* n_dev, int32_t N, const ViewsArg& va, uint32_t* tiles, uint32_t* emit_g,
                          uint32_t* inst_off,
                          bool all_off, uint32_t* block_start, bool starts_marked, int64_t capacity,
                          uint32_t* overflow, hipStream_t s) {
  const int64_t n = (int64_t)va.n * N;
  if (n <= 0 || capacity <= 0) return hipSuccess;
  if (!starts_marked)
    hipLaunchKernelGGL(k_block_starts, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, offsets, n_dev, n, capacity,
                       block_start);
  hipLaunchKernelGGL(k_dup_lb, dim3((unsigned)((capacity + kLb - 1) / kLb)), dim3(kLbThreads), 0, s, rec, order, offsets,
                     counts, block_start, n_dev, n, N, va, capacity, tiles, emit_g, inst_off, all_off ? 1 : 0,
                     overflow);
  return hipGetLastError();
}

// Gaussian index of every instance in blend order.
__global__ void __launch_bounds__(256)
k_gather_g(const uint32_t* __restrict__ vals, const uint32_t* __restrict__ emit_g, const uint32_t* __restrict__ n_dev,
           int64_t cap, uint32_t* __restrict__ out) {
  const int64_t n = sort_count(n_dev, cap), step = (int64_t)gridDim.x * 256;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += step) out[i] = emit_g[vals[i]];
}

hipError_t gather_gaussians(const uint32_t* vals, const uint32_t* emit_g, const uint32_t* n_dev, int64_t cap,
                            uint32_t* out, hipStream_t s) {
  if (cap <= 0) return hipSuccess;
  // (a launch holds less than 2^32 lanes)
  const int64_t blocks = std::min<int64_t>((cap + 255) / 256, int64_t(1) << 23);
  hipLaunchKernelGGL(k_gather_g, dim3((unsigned)blocks), dim3(256), 0, s, vals, emit_g, n_dev, cap, out);
  return hipGetLastError();
}

// ---------------------------------------------------------------------- ranges
// Four consecutive instances per lane (one 16-B load when they are all present, the tile
// arrays being 16-B aligned), each compared with its predecessor.
constexpr int kRangePer = 4;

__global__ void __launch_bounds__(256)
k_ranges(const uint32_t* __restrict__ tiles, const uint32_t* __restrict__ n_dev, int64_t cap,
         uint2* __restrict__ ranges, uint32_t n_tiles) {
  const int64_t i0 = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * kRangePer;
  const uint32_t n = sort_count(n_dev, cap);
  if (i0 >= n) return;
  uint32_t t[kRangePer];
  if (i0 + kRangePer <= n) {
    const uint4 q = *(const uint4*)(tiles + i0);
    t[0] = q.x; t[1] = q.y; t[2] = q.z; t[3] = q.w;
  } else {
#pragma unroll
    for (int k = 0; k < kRangePer; ++k) t[k] = i0 + k < n ? tiles[i0 + k] : 0xffffffffu;
  }
  uint32_t tp = i0 > 0 ? tiles[i0 - 1] : 0xffffffffu;
#pragma unroll
  for (int k = 0; k < kRangePer; ++k) {
    const int64_t i = i0 + k;
    if (i >= n) break;
    if (i == 0) {
      if (t[k] < n_tiles) ranges[t[k]].x = 0;
    } else if (tp != t[k]) {
      if (tp < n_tiles) ranges[tp].y = (uint32_t)i;
      if (t[k] < n_tiles) ranges[t[k]].x = (uint32_t)i;
    }
    if (i == (int64_t)n - 1 && t[k] < n_tiles) ranges[t[k]].y = n;
    tp = t[k];
  }
}

hipError_t tile_ranges(const uint32_t* tiles, const uint32_t* n_dev, int64_t cap, uint2* ranges, int64_t n_tiles,
                       hipStream_t s) {
  if (cap <= 0) return hipSuccess;
  const int64_t lanes = (cap + kRangePer - 1) / kRangePer;
  hipLaunchKernelGGL(k_ranges, dim3((unsigned)((lanes + 255) / 256)), dim3(256), 0, s, tiles, n_dev, cap, ranges,
                     (uint32_t)n_tiles);
  return hipGetLastError();
}

}  // namespace gs
