// Particle binning: cell keys, a stable LSD radix sort of (key, index) pairs,
// the bin offset array, and permutation gathers/scatters.
//
// This is the GPU form of the paper's local particle ordering (Sec. 3.3.1,
// "Ordering the particles locally"): particles of one group are stored
// contiguously, groups in increasing order, with an offset array of size
// groups+1 whose last entry is the particle count.  The paper partitions by
// x3 slice with an incomplete Quicksort; here a group is a window of W cell
// layers of a T x T tile column (x3 fastest within a column, as the paper's
// slices), and the partition is a stable radix sort, so that ties keep their
// input order and the result is reproducible bit for bit.
#include "device_common.h"
#include "launch.h"

namespace ptk {

// ---------------------------------------------------------------------------
// keys and locate
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint32_t key_of(const double* __restrict__ X, int64_t i, int N, double invd,
                                           const BinGeom& g, int* __restrict__ flag) {
  double x1 = X[3 * i], x2 = X[3 * i + 1], x3 = X[3 * i + 2];
  if (!in_domain3(x1, x2, x3)) {
    raise_flag(flag, kFlagDomain);
    return 0;
  }
  int c1, c2, c3;
  double t;
  locate(x1, N, invd, &c1, &t);
  locate(x2, N, invd, &c2, &t);
  locate(x3, N, invd, &c3, &t);
  return bin_key(c1, c2, c3, g);
}

__global__ __launch_bounds__(256) void k_keys(const double* __restrict__ X, int64_t n, int N,
                                              double invd, BinGeom g, uint32_t* __restrict__ keys,
                                              int* __restrict__ flag) {
  int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) keys[i] = key_of(X, i, N, invd, g, flag);
}

__global__ __launch_bounds__(256) void k_locate(const double* __restrict__ X, int64_t n3, int N,
                                                double invd, int32_t* __restrict__ cell,
                                                double* __restrict__ off, int* __restrict__ flag) {
  int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n3) return;
  double x = X[i];
  if (!in_domain(x)) {
    raise_flag(flag, kFlagDomain);
    cell[i] = 0;
    if (off) off[i] = 0.0;
    return;
  }
  int c;
  double t;
  locate(x, N, invd, &c, &t);
  cell[i] = c;
  if (off) off[i] = t;
}

// ---------------------------------------------------------------------------
// stable LSD radix sort, one pass per digit
//   tile = 256 threads x 8 items; each wave owns 512 consecutive items and
//   ranks them in 8 rounds of 64 with a ballot-built "same digit" lane mask.
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint32_t block_excl_scan_256(uint32_t v, uint32_t* sh, uint32_t* total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t x = v;
  for (int o = 1; o < 64; o <<= 1) {
    uint32_t y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  if (lane == 63) sh[wave] = x;
  __syncthreads();
  uint32_t wpre = 0, tot = 0;
  for (int w = 0; w < 4; ++w) {
    if (w < wave) wpre += sh[w];
    tot += sh[w];
  }
  __syncthreads();
  *total = tot;
  return wpre + x - v;
}

constexpr int kSortThreads = 256;
constexpr int kSortItems = 8;
constexpr int kTile = kSortThreads * kSortItems;  // 2048

// tiles of a sort of n elements, or of min(n, *n_dev) when the count lives on
// the device; the digit histograms are laid out [digit][tiles]
__device__ __forceinline__ int64_t sort_tiles(int64_t n, const uint32_t* n_dev) {
  if (n_dev) n = min(n, (int64_t)*n_dev);
  return (n + kTile - 1) / kTile;
}

// keys and, of the same tiles, the histogram of the sort's first digit
__global__ __launch_bounds__(256) void k_keys_hist(const double* __restrict__ X, int64_t n, int N, double invd,
                                                   BinGeom g, uint32_t mask, uint32_t* __restrict__ keys,
                                                   uint32_t* __restrict__ hist, int64_t n_tiles,
                                                   int* __restrict__ flag) {
  __shared__ uint32_t h[256];
  h[threadIdx.x] = 0;
  __syncthreads();
  const int64_t base = (int64_t)blockIdx.x * kTile;
  for (int k = 0; k < kSortItems; ++k) {
    const int64_t i = base + k * kSortThreads + threadIdx.x;
    if (i < n) {
      const uint32_t key = key_of(X, i, N, invd, g, flag);
      keys[i] = key;
      atomicAdd(&h[key & mask], 1u);
    }
  }
  __syncthreads();
  if (threadIdx.x <= mask) hist[(int64_t)threadIdx.x * n_tiles + blockIdx.x] = h[threadIdx.x];
}

// n_dev (optional, here and below): the element count held on the device; n is
// then an upper bound that sized the grid, and tiles past the count contribute
// nothing.
__global__ __launch_bounds__(256) void k_radix_hist(const uint32_t* __restrict__ keys, int64_t n,
                                                    const uint32_t* __restrict__ n_dev, int shift, uint32_t mask,
                                                    uint32_t* __restrict__ hist, int64_t n_tiles) {
  if (n_dev) {
    n_tiles = sort_tiles(n, n_dev);
    if ((int64_t)blockIdx.x >= n_tiles) return;
    n = min(n, (int64_t)*n_dev);
  }
  __shared__ uint32_t h[256];
  h[threadIdx.x] = 0;
  __syncthreads();
  const int64_t base = (int64_t)blockIdx.x * kTile;
  for (int k = 0; k < kSortItems; ++k) {
    int64_t i = base + k * kSortThreads + threadIdx.x;
    if (i < n) atomicAdd(&h[(keys[i] >> shift) & mask], 1u);
  }
  __syncthreads();
  if (threadIdx.x <= mask) hist[(int64_t)threadIdx.x * n_tiles + blockIdx.x] = h[threadIdx.x];
}

// incl: the histogram rows after k_scan_rows, so a row's last entry is its
// digit's count; the digits' starts are those counts' scan, done here by every
// block
__global__ __launch_bounds__(256) void k_radix_scatter(
    const uint32_t* __restrict__ keys_in, const uint32_t* __restrict__ vals_in, int64_t n,
    const uint32_t* __restrict__ n_dev, int shift, uint32_t mask, int bits, const uint32_t* __restrict__ incl,
    int64_t n_tiles, uint32_t* __restrict__ keys_out, uint32_t* __restrict__ vals_out) {
  if (n_dev) {
    n_tiles = sort_tiles(n, n_dev);
    n = min(n, (int64_t)*n_dev);
  }
  if ((int64_t)blockIdx.x * kTile >= n) return;
  __shared__ uint32_t wcount[4][256];
  __shared__ uint32_t dstart[256], dpos[256];
  __shared__ uint32_t scan_sh[4];
  __shared__ uint32_t skey[kTile], sval[kTile];
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  for (int d = threadIdx.x; d < 4 * 256; d += 256) (&wcount[0][0])[d] = 0;
  uint32_t dcount = 0, dbefore = 0;  // of digit threadIdx.x: its count, and that of the tiles before this one
  if (threadIdx.x <= mask) {
    const uint32_t* row = incl + (int64_t)threadIdx.x * n_tiles;
    dcount = row[n_tiles - 1];
    dbefore = blockIdx.x ? row[(int64_t)blockIdx.x - 1] : 0u;
  }
  __syncthreads();
  const int64_t wbase = (int64_t)blockIdx.x * kTile + wave * (64 * kSortItems);
  const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  uint32_t key[kSortItems], val[kSortItems], rank[kSortItems];
  for (int r = 0; r < kSortItems; ++r) {
    int64_t i = wbase + r * 64 + lane;
    bool valid = i < n;
    uint32_t k = valid ? keys_in[i] : 0u;
    uint32_t v = valid ? (vals_in ? vals_in[i] : (uint32_t)i) : 0u;
    uint32_t d = (k >> shift) & mask;
    uint64_t peers = __ballot(valid);
    for (int b = 0; b < bits; ++b) {
      uint64_t m = __ballot((d >> b) & 1u);
      peers &= ((d >> b) & 1u) ? m : ~m;
    }
    uint32_t before = (uint32_t)__popcll(peers & lt_mask);
    uint32_t base = valid ? wcount[wave][d] : 0u;
    // every lane of this wave has read the running count before the leader of
    // each digit group adds the group's size
    __builtin_amdgcn_wave_barrier();
    if (valid && before == 0) wcount[wave][d] = base + (uint32_t)__popcll(peers);
    __builtin_amdgcn_wave_barrier();
    key[r] = k;
    val[r] = v;
    rank[r] = valid ? base + before : 0xFFFFFFFFu;
  }
  __syncthreads();
  // exclusive prefix of the per-wave counts over waves, per digit, and the
  // start of each digit's run inside the tile
  uint32_t tile_count = 0;
  {
    for (int w = 0; w < 4; ++w) {
      uint32_t c = wcount[w][threadIdx.x];
      wcount[w][threadIdx.x] = tile_count;
      tile_count += c;
    }
  }
  uint32_t ntile;
  const uint32_t my_start = block_excl_scan_256(tile_count, scan_sh, &ntile);
  uint32_t all;
  dstart[threadIdx.x] = my_start;
  dpos[threadIdx.x] = block_excl_scan_256(dcount, scan_sh, &all) + dbefore - my_start;
  __syncthreads();
  // the tile in digit order in LDS, then written out run by run: consecutive
  // threads write consecutive addresses of a digit's run
  for (int r = 0; r < kSortItems; ++r) {
    if (rank[r] == 0xFFFFFFFFu) continue;
    const uint32_t d = (key[r] >> shift) & mask;
    const uint32_t lp = dstart[d] + wcount[wave][d] + rank[r];
    skey[lp] = key[r];
    sval[lp] = val[r];
  }
  __syncthreads();
  for (uint32_t j = threadIdx.x; j < ntile; j += kSortThreads) {
    const uint32_t k = skey[j];
    const uint32_t pos = dpos[(k >> shift) & mask] + j;
    keys_out[pos] = k;
    vals_out[pos] = sval[j];
  }
}

// In-place inclusive scan of every row of a [rows][len] array, a block a row:
// the histogram rows of a sort pass, or the movers per tile.  One launch where
// a scan of the whole array takes three (block sums, their scan, the sums
// added), and no work for digits that do not occur: what these launches cost
// is their latency.  (Re-binning is 12 launches with two digits, 23 before; a
// Heun step of 10^6 particles with axes at 256^3 and a store 975 us, now 904;
// the sort of a call with 1.25e7 at 512^3, whose first histogram is now taken
// with the keys, about 50 us less: learned inference 2903 us, now 2852.)
constexpr int kScanThreads = 1024;

__global__ __launch_bounds__(1024) void k_scan_rows(uint32_t* __restrict__ a, int64_t len, int64_t n,
                                                    const uint32_t* __restrict__ n_dev) {
  if (n_dev) len = sort_tiles(n, n_dev);
  constexpr int W = kScanThreads / 64;
  __shared__ uint32_t sh[2][W];
  uint32_t* row = a + (int64_t)blockIdx.x * len;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t carry = 0;
  int buf = 0;
  for (int64_t base = 0; base < len; base += 4 * kScanThreads, buf ^= 1) {
    const int64_t i = base + 4 * (int64_t)threadIdx.x;
    uint32_t v[4];
    for (int k = 0; k < 4; ++k) v[k] = i + k < len ? row[i + k] : 0u;
    for (int k = 1; k < 4; ++k) v[k] += v[k - 1];
    uint32_t x = v[3];
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t y = __shfl_up(x, o, 64);
      if (lane >= o) x += y;
    }
    if (lane == 63) sh[buf][wave] = x;
    __syncthreads();  // (the buffer is written again two rounds on, past the next barrier)
    uint32_t before = carry + x - v[3];
    for (int w = 0; w < W; ++w) {
      const uint32_t t = sh[buf][w];
      if (w < wave) before += t;
      carry += t;
    }
    for (int k = 0; k < 4; ++k)
      if (i + k < len) row[i + k] = before + v[k];
  }
}

// offsets[b] = first sorted index with key >= b, for b in [0, n_bins]
__global__ __launch_bounds__(256) void k_offsets(const uint32_t* __restrict__ skeys, int64_t n, int64_t n_bins,
                                                 uint32_t* __restrict__ offsets, const uint32_t* __restrict__ perm,
                                                 uint32_t* __restrict__ unsorted) {
  int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i > n) return;
  if (unsorted && i < n) unsorted[perm[i]] = skeys[i];
  int64_t lo = (i == 0) ? -1 : (int64_t)skeys[i - 1];
  int64_t hi = (i == n) ? n_bins : (int64_t)skeys[i];
  if (hi > n_bins) hi = n_bins;  // keys are < n_bins by construction; never write past the array
  for (int64_t b = lo + 1; b <= hi; ++b) offsets[b] = (uint32_t)i;
}

// Rows of W elements between orders.  A block takes 256 rows: their indices go
// through LDS, then consecutive threads take consecutive elements, so a row at
// a scattered place is one contiguous access of neighbouring lanes and the
// memory pipeline sees one segment per row.  (A thread per row issues W
// accesses of 64 scattered segments each instead: a resident Heun step and
// store of 10^8 particles at 1024^3 49.1 ms, now 47.4; five AB2 steps and a
// store of 10^7 at 256^3 8.00 ms, now 7.31.)
constexpr int kRowBlock = 256;

template <typename T>
__global__ __launch_bounds__(256) void k_gather3(const T* __restrict__ in, const uint32_t* __restrict__ perm,
                                                 int64_t n, T* __restrict__ out) {
  __shared__ uint32_t rows[kRowBlock];
  const int64_t base = (int64_t)blockIdx.x * kRowBlock;
  const int nb = (int)min((int64_t)kRowBlock, n - base);
  rows[threadIdx.x] = (int)threadIdx.x < nb ? perm[base + threadIdx.x] : 0u;
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    const int e = i * kRowBlock + threadIdx.x, r = e / 3;
    if (r < nb) out[3 * base + e] = in[3 * (int64_t)rows[r] + (e - 3 * r)];
  }
}

template <typename T, int W>
__global__ __launch_bounds__(256) void k_scatter(const T* __restrict__ in, const uint32_t* __restrict__ idx,
                                                 int64_t n, T* __restrict__ out) {
  __shared__ uint32_t rows[kRowBlock];
  const int64_t base = (int64_t)blockIdx.x * kRowBlock;
  const int nb = (int)min((int64_t)kRowBlock, n - base);
  rows[threadIdx.x] = (int)threadIdx.x < nb ? idx[base + threadIdx.x] : 0u;
  __syncthreads();
#pragma unroll
  for (int i = 0; i < W; ++i) {
    const int e = i * kRowBlock + threadIdx.x, r = e / W;
    if (r < nb) out[W * (int64_t)rows[r] + (e - W * r)] = in[W * base + e];
  }
}

// out[idx[k]] = in[src[k]] for rows of 3: a gather and a scatter without the
// array between them
__global__ __launch_bounds__(256) void k_move3(const double* __restrict__ in, const uint32_t* __restrict__ src,
                                               const uint32_t* __restrict__ idx, int64_t n,
                                               double* __restrict__ out) {
  __shared__ uint32_t from[kRowBlock], to[kRowBlock];
  const int64_t base = (int64_t)blockIdx.x * kRowBlock;
  const int nb = (int)min((int64_t)kRowBlock, n - base);
  from[threadIdx.x] = (int)threadIdx.x < nb ? src[base + threadIdx.x] : 0u;
  to[threadIdx.x] = (int)threadIdx.x < nb ? idx[base + threadIdx.x] : 0u;
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    const int e = i * kRowBlock + threadIdx.x, r = e / 3, c = e - 3 * r;
    if (r < nb) out[3 * (int64_t)to[r] + c] = in[3 * (int64_t)from[r] + c];
  }
}

__global__ __launch_bounds__(256) void k_gather_u32(const uint32_t* __restrict__ in,
                                                    const uint32_t* __restrict__ perm, int64_t n,
                                                    uint32_t* __restrict__ out) {
  int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (k >= n) return;
  out[k] = in[perm[k]];
}

// ---------------------------------------------------------------------------
// incremental re-binning (particles move less than a cell per step, so few
// change bins; only those are sorted, the rest keep their relative order)
// ---------------------------------------------------------------------------
// Tile of 2048 items: wave w owns items [512w, 512w + 512) of the tile in 8
// rounds of 64.  For each item: whether its key changed ("mover") and the
// number of movers before it in the tile.
struct TileMovers {
  uint32_t ok[kSortItems], nk[kSortItems], before[kSortItems];
  bool valid[kSortItems], mover[kSortItems];
  uint32_t total;
};

__device__ __forceinline__ void tile_movers(const uint32_t* okeys, const uint32_t* nkeys, int64_t n, TileMovers& t) {
  __shared__ uint32_t wsum[4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t wbase = (int64_t)blockIdx.x * kTile + wave * (64 * kSortItems);
  const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  uint32_t run = 0;
  for (int r = 0; r < kSortItems; ++r) {
    const int64_t i = wbase + r * 64 + lane;
    t.valid[r] = i < n;
    t.ok[r] = t.valid[r] ? okeys[i] : 0u;
    t.nk[r] = t.valid[r] ? nkeys[i] : 0u;
    t.mover[r] = t.valid[r] && t.ok[r] != t.nk[r];
    const uint64_t bal = __ballot(t.mover[r]);
    t.before[r] = run + (uint32_t)__popcll(bal & lt_mask);
    run += (uint32_t)__popcll(bal);
  }
  if (lane == 0) wsum[wave] = run;
  __syncthreads();
  uint32_t pre = 0, tot = 0;
  for (int w = 0; w < 4; ++w) {
    if (w < wave) pre += wsum[w];
    tot += wsum[w];
  }
  for (int r = 0; r < kSortItems; ++r) t.before[r] += pre;
  t.total = tot;
}

__device__ __forceinline__ int64_t tile_item(int r) {
  return (int64_t)blockIdx.x * kTile + (threadIdx.x >> 6) * (64 * kSortItems) + r * 64 + (threadIdx.x & 63);
}

// movers per tile
__global__ __launch_bounds__(256) void k_rebin_count(const uint32_t* __restrict__ okeys,
                                                     const uint32_t* __restrict__ nkeys, int64_t n,
                                                     uint32_t* __restrict__ tile_cnt) {
  TileMovers t;
  tile_movers(okeys, nkeys, n, t);
  if (threadIdx.x == 0) tile_cnt[blockIdx.x] = t.total;
}

// movers, in current order, to (mk, mv, mo) = (new key, current index, old key)
__global__ __launch_bounds__(256) void k_rebin_compact(const uint32_t* __restrict__ okeys,
                                                       const uint32_t* __restrict__ nkeys, int64_t n,
                                                       const uint32_t* __restrict__ tile_off,
                                                       uint32_t* __restrict__ mk, uint32_t* __restrict__ mv,
                                                       uint32_t* __restrict__ mo) {
  TileMovers t;
  tile_movers(okeys, nkeys, n, t);
  const uint32_t base = blockIdx.x ? tile_off[blockIdx.x - 1] : 0u;
  for (int r = 0; r < kSortItems; ++r)
    if (t.mover[r]) {
      mk[base + t.before[r]] = t.nk[r];
      mv[base + t.before[r]] = (uint32_t)tile_item(r);
      mo[base + t.before[r]] = t.ok[r];
    }
}

// first index i < m with keys[i] >= b (m if none), for sorted keys
__device__ __forceinline__ uint32_t first_ge(const uint32_t* __restrict__ keys, uint32_t m, uint32_t b) {
  uint32_t lo = 0, hi = m;
  while (lo < hi) {
    const uint32_t mid = lo + (hi - lo) / 2;
    if (keys[mid] < b)
      lo = mid + 1;
    else
      hi = mid;
  }
  return lo;
}

// Per bin b = 0..n_bins: the movers whose old key < b (mo: their old keys, in
// current order, so sorted) and those whose new key < b (sk: sorted), by binary
// search (one thread per bin, so the cost does not depend on how the keys are
// spread; m is read on the device); the new offset: elements with new key < b
// = (old key < b) - (movers whose old key < b) + (movers whose new key < b);
// and the cleared count of movers that come from earlier bins.
__global__ __launch_bounds__(256) void k_rebin_offsets(const uint32_t* __restrict__ mo,
                                                       const uint32_t* __restrict__ sk,
                                                       const uint32_t* __restrict__ m_dev,
                                                       const uint32_t* __restrict__ ooff, int64_t n_bins,
                                                       uint32_t* __restrict__ out_before,
                                                       uint32_t* __restrict__ in_start, uint32_t* __restrict__ noff,
                                                       uint32_t* __restrict__ inc_before) {
  const int64_t b = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (b > n_bins) return;
  const uint32_t m = *m_dev;
  const uint32_t out = first_ge(mo, m, (uint32_t)b), in = first_ge(sk, m, (uint32_t)b);
  out_before[b] = out;
  in_start[b] = in;
  noff[b] = ooff[b] - out + in;
  inc_before[b] = 0u;
}

// Place the movers, sorted by (new key, current index): in bin b they follow
// the movers from earlier bins and, if they come from a later bin, the
// particles that stay in b.  Also counts, per bin, the movers from earlier bins.
__global__ __launch_bounds__(256) void k_rebin_movers(const uint32_t* __restrict__ sk, const uint32_t* __restrict__ sv,
                                                      const uint32_t* __restrict__ m_dev,
                                                      const uint32_t* __restrict__ ooff,
                                                      const uint32_t* __restrict__ noff,
                                                      const uint32_t* __restrict__ in_start,
                                                      const uint32_t* __restrict__ out_before,
                                                      uint32_t* __restrict__ inc_before, uint32_t* __restrict__ perm,
                                                      uint32_t* __restrict__ skeys) {
  const int64_t m = *m_dev;
  for (int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x; r < m; r += (int64_t)gridDim.x * 256) {
    const uint32_t b = sk[r], i = sv[r];
    const bool from_before = i < ooff[b];
    if (from_before) atomicAdd(&inc_before[b], 1u);
    const uint32_t stay = (ooff[b + 1] - ooff[b]) - (out_before[b + 1] - out_before[b]);
    const uint32_t pos = noff[b] + (uint32_t)(r - in_start[b]) + (from_before ? 0u : stay);
    perm[pos] = i;
    skeys[pos] = b;
  }
}

// Place the particles that stay in their bin b: after the movers from earlier
// bins, in their current order.
__global__ __launch_bounds__(256) void k_rebin_stayers(const uint32_t* __restrict__ okeys,
                                                       const uint32_t* __restrict__ nkeys, int64_t n,
                                                       const uint32_t* __restrict__ tile_off,
                                                       const uint32_t* __restrict__ ooff,
                                                       const uint32_t* __restrict__ noff,
                                                       const uint32_t* __restrict__ out_before,
                                                       const uint32_t* __restrict__ inc_before,
                                                       uint32_t* __restrict__ perm, uint32_t* __restrict__ skeys) {
  TileMovers t;
  tile_movers(okeys, nkeys, n, t);
  const uint32_t base = blockIdx.x ? tile_off[blockIdx.x - 1] : 0u;
  for (int r = 0; r < kSortItems; ++r) {
    if (!t.valid[r] || t.mover[r]) continue;
    const uint32_t b = t.nk[r];
    const uint32_t i = (uint32_t)tile_item(r);
    const uint32_t movers_before = base + t.before[r];         // movers at positions < i
    const uint32_t out_in_seg = movers_before - out_before[b];  // of them, inside bin b's segment
    const uint32_t pos = noff[b] + inc_before[b] + (i - ooff[b]) - out_in_seg;
    perm[pos] = i;
    skeys[pos] = b;
  }
}

// ---------------------------------------------------------------------------
// host launchers
// ---------------------------------------------------------------------------
static inline unsigned blocks_for(int64_t n, int per) { return (unsigned)((n + per - 1) / per); }

// passes of a sort of keys below 2^key_bits, and the bits of a digit
static inline int sort_passes(int key_bits) { return key_bits <= 0 ? 1 : (key_bits + 7) / 8; }
static inline int digit_bits(int key_bits) {
  const int passes = sort_passes(key_bits);
  return key_bits <= 0 ? 1 : (key_bits + passes - 1) / passes;
}

hipError_t launch_keys(const double* X, int64_t n, int N, double invd, const BinGeom& g, uint32_t* keys,
                       int* flag, hipStream_t s) {
  if (n == 0) return hipSuccess;
  k_keys<<<blocks_for(n, 256), 256, 0, s>>>(X, n, N, invd, g, keys, flag);
  return hipGetLastError();
}

hipError_t launch_keys_hist(const double* X, int64_t n, int N, double invd, const BinGeom& g, int key_bits,
                            uint32_t* keys, uint32_t* hist, int* flag, hipStream_t s) {
  if (n == 0) return hipSuccess;
  const unsigned n_tiles = blocks_for(n, kTile);
  k_keys_hist<<<n_tiles, 256, 0, s>>>(X, n, N, invd, g, (1u << digit_bits(key_bits)) - 1u, keys, hist,
                                      (int64_t)n_tiles, flag);
  return hipGetLastError();
}

hipError_t launch_locate(const double* X, int64_t n3, int N, double invd, int32_t* cell, double* off,
                         int* flag, hipStream_t s) {
  if (n3 == 0) return hipSuccess;
  k_locate<<<blocks_for(n3, 256), 256, 0, s>>>(X, n3, N, invd, cell, off, flag);
  return hipGetLastError();
}

size_t sort_hist_words(int64_t n) {
  int64_t n_tiles = (n + kTile - 1) / kTile;
  return (size_t)256 * (size_t)(n_tiles > 0 ? n_tiles : 1);
}

// Stable sort of keys.  Values: those in va if vals_in_va, else the input
// positions.  n_dev (optional) holds the element count on the device, n an
// upper bound.  have_hist: hist holds the first digit's histogram already
// (launch_keys_hist).  On return *keys_sorted and *perm point into {ka, kb} / {va, vb}.
hipError_t radix_sort_keys(uint32_t* ka, uint32_t* kb, uint32_t* va, uint32_t* vb, int64_t n,
                           const uint32_t* n_dev, bool vals_in_va, int key_bits, uint32_t* hist, bool have_hist,
                           uint32_t** keys_sorted, uint32_t** perm, hipStream_t s) {
  if (n == 0) {
    *keys_sorted = ka;
    *perm = va;
    return hipSuccess;
  }
  const int64_t n_tiles = (n + kTile - 1) / kTile;
  const int passes = sort_passes(key_bits);
  const int bits = digit_bits(key_bits);
  const uint32_t mask = (1u << bits) - 1u;
  // pass p reads (kin, vin) and writes (kout, vout); the first pass takes the
  // input positions as values
  uint32_t *kin = ka, *kout = kb, *vin = vals_in_va ? va : nullptr, *vout = vals_in_va ? vb : va,
           *vspare = vb;
  for (int p = 0; p < passes; ++p) {
    const int shift = p * bits;
    if (p > 0 || !have_hist)
      k_radix_hist<<<(unsigned)n_tiles, 256, 0, s>>>(kin, n, n_dev, shift, mask, hist, n_tiles);
    // with the count on the device, every kernel sizes the histogram from it
    k_scan_rows<<<mask + 1u, kScanThreads, 0, s>>>(hist, n_tiles, n, n_dev);
    k_radix_scatter<<<(unsigned)n_tiles, 256, 0, s>>>(kin, vin, n, n_dev, shift, mask, bits, hist, n_tiles,
                                                      kout, vout);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    uint32_t* t = kin;
    kin = kout;
    kout = t;
    uint32_t* old_vin = vin;
    vin = vout;
    vout = old_vin ? old_vin : vspare;
  }
  *keys_sorted = kin;
  *perm = vin;
  return hipSuccess;
}

size_t rebin_block_words(int64_t n) { return (size_t)((n + kTile - 1) / kTile + 2); }

hipError_t rebin_incremental(const uint32_t* okeys, const uint32_t* ooff, const uint32_t* nkeys, int64_t n,
                             int64_t n_bins, int key_bits, const RebinScratch& w, uint32_t* perm, uint32_t* skeys,
                             uint32_t* noff, hipStream_t s) {
  if (n == 0) return hipSuccess;
  const int64_t n_tiles = (n + kTile - 1) / kTile;
  hipError_t e;
  // movers per tile, inclusive scan: the last entry becomes the mover count m
  k_rebin_count<<<(unsigned)n_tiles, 256, 0, s>>>(okeys, nkeys, n, w.blockoff);
  k_scan_rows<<<1, kScanThreads, 0, s>>>(w.blockoff, n_tiles, 0, nullptr);
  const uint32_t* m_dev = w.blockoff + (n_tiles - 1);
  // movers in current order (their old keys are then sorted), then sorted by new key
  k_rebin_compact<<<(unsigned)n_tiles, 256, 0, s>>>(okeys, nkeys, n, w.blockoff, w.mk_a, w.mv_a, w.mo);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  uint32_t *sk = nullptr, *sv = nullptr;
  if ((e = radix_sort_keys(w.mk_a, w.mk_b, w.mv_a, w.mv_b, n, m_dev, true, key_bits, w.hist, false, &sk, &sv, s)) !=
      hipSuccess)
    return e;
  k_rebin_offsets<<<blocks_for(n_bins + 1, 256), 256, 0, s>>>(w.mo, sk, m_dev, ooff, n_bins, w.out_before, w.in_start,
                                                             noff, w.inc_before);
  const int64_t mgrid = min((int64_t)4096, (n + 255) / 256);
  k_rebin_movers<<<(unsigned)mgrid, 256, 0, s>>>(sk, sv, m_dev, ooff, noff, w.in_start, w.out_before, w.inc_before,
                                                 perm, skeys);
  k_rebin_stayers<<<(unsigned)n_tiles, 256, 0, s>>>(okeys, nkeys, n, w.blockoff, ooff, noff, w.out_before,
                                                    w.inc_before, perm, skeys);
  return hipGetLastError();
}

__global__ __launch_bounds__(256) void k_iota(uint32_t* __restrict__ p, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) p[i] = (uint32_t)i;
}

hipError_t launch_iota(uint32_t* p, int64_t n, hipStream_t s) {
  if (n == 0) return hipSuccess;
  k_iota<<<blocks_for(n, 256), 256, 0, s>>>(p, n);
  return hipGetLastError();
}

hipError_t launch_offsets(const uint32_t* skeys, int64_t n, int64_t n_bins, uint32_t* offsets, hipStream_t s,
                          const uint32_t* perm, uint32_t* unsorted) {
  k_offsets<<<blocks_for(n + 1, 256), 256, 0, s>>>(skeys, n, n_bins, offsets, perm, unsorted);
  return hipGetLastError();
}

hipError_t gather3_f64(const double* in, const uint32_t* perm, int64_t n, double* out, hipStream_t s) {
  if (n == 0) return hipSuccess;
  k_gather3<double><<<blocks_for(n, 256), 256, 0, s>>>(in, perm, n, out);
  return hipGetLastError();
}

hipError_t gather3_f32(const float* in, const uint32_t* perm, int64_t n, float* out, hipStream_t s) {
  if (n == 0) return hipSuccess;
  k_gather3<float><<<blocks_for(n, 256), 256, 0, s>>>(in, perm, n, out);
  return hipGetLastError();
}

hipError_t gather_u32(const uint32_t* in, const uint32_t* perm, int64_t n, uint32_t* out, hipStream_t s) {
  if (n == 0) return hipSuccess;
  k_gather_u32<<<blocks_for(n, 256), 256, 0, s>>>(in, perm, n, out);
  return hipGetLastError();
}

template <typename T>
static hipError_t scatter_rows(const T* in, const uint32_t* idx, int64_t n, int width, T* out, hipStream_t s) {
  if (n == 0) return hipSuccess;
  const unsigned blocks = blocks_for(n, kRowBlock);
  if (width == 3)
    k_scatter<T, 3><<<blocks, 256, 0, s>>>(in, idx, n, out);
  else if (width == 9)
    k_scatter<T, 9><<<blocks, 256, 0, s>>>(in, idx, n, out);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t scatter_f64(const double* in, const uint32_t* idx, int64_t n, int width, double* out,
                       hipStream_t s) {
  return scatter_rows(in, idx, n, width, out, s);
}

hipError_t scatter_f32(const float* in, const uint32_t* idx, int64_t n, int width, float* out,
                       hipStream_t s) {
  return scatter_rows(in, idx, n, width, out, s);
}

hipError_t move3_f64(const double* in, const uint32_t* src, const uint32_t* idx, int64_t n, double* out,
                     hipStream_t s) {
  if (n == 0) return hipSuccess;
  k_move3<<<blocks_for(n, kRowBlock), 256, 0, s>>>(in, src, idx, n, out);
  return hipGetLastError();
}

}  // namespace ptk
