// Segmented, stable sort of (uint32 key, uint32 value) pairs: LSD radix passes for the segments too large to be sorted
// in runs, and the merge of the others' runs (block_sort.h sorts a run).
//
// Segments are contiguous ranges sorted independently (frames when building
// the voxel structure, edges when binning source points per iteration); they
// are known on the host, so the tile -> segment table is static and every
// launch has a fixed shape.  Each 8-bit digit takes two kernels:
//   hist    per tile, a 256-bin digit histogram (LDS atomics); the caller's
//           key kernel has written the first digit's
//   scatter per tile, the tile's first slot of every digit (its segment's
//           histograms summed, one digit per thread) and stable ranks (in
//           the wavefronts from ballots, block_sort.h), keys and values to
//           their slots.
// Segments of more than kFusedTiles tiles have their histograms scanned by a
// kernel of their own before the scatter: a tile would otherwise read the
// whole segment's histograms (1 KB per tile of the segment).
//
// The sort is bound by its dependent launches and barriers, not by bytes:
// ranks taken per wavefront over eight rounds need 5 barriers per tile where
// ranks per block of 256 items needed 32, and every load of a tile is issued
// at once.  8 frames x 30,000 points, 28 edges (420 tiles): scatter and scan
// 11.9 + 8.0 -> 9.3 us per digit.
#include "block_sort.h"

namespace rkhsba {
namespace {

constexpr int kFusedTiles = 64;

__global__ __launch_bounds__(kSortThreads) void k_hist(const uint32_t* __restrict__ keys,
                                                       const SortTile* __restrict__ tiles, int shift,
                                                       uint32_t* __restrict__ hist) {
  __shared__ uint32_t h[256];
  const int tid = threadIdx.x;
  h[tid] = 0;
  const SortTile t = tiles[blockIdx.x];
  uint32_t key[kSortItems];
#pragma unroll
  for (int r = 0; r < kSortItems; ++r) {
    const int k = r * kSortThreads + tid;
    key[r] = k < t.count ? keys[t.start + k] : 0u;
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kSortItems; ++r)
    if (r * kSortThreads + tid < t.count) atomicAdd(&h[(key[r] >> shift) & 0xffu], 1u);
  __syncthreads();
  hist[(int64_t)blockIdx.x * 256 + tid] = h[tid];
}

__global__ __launch_bounds__(256) void k_scan(uint32_t* __restrict__ hist, const SortSeg* __restrict__ segs) {
  __shared__ uint32_t wtot[4];
  const int d = threadIdx.x;
  const SortSeg s = segs[blockIdx.x];
  if (s.n_tiles == 0) return;  // (uniform) sorted in runs
  uint32_t run = 0;
  for (int t = 0; t < s.n_tiles; ++t) {
    uint32_t* h = hist + (int64_t)(s.tile0 + t) * 256 + d;
    const uint32_t c = *h;
    *h = run;  // offset of this tile's first key of digit d among the segment's digit-d keys
    run += c;
  }
  const uint32_t base = digit_exclusive_scan(run, wtot);
  for (int t = 0; t < s.n_tiles; ++t) hist[(int64_t)(s.tile0 + t) * 256 + d] += base;
}

// FUSED: hist holds the tiles' digit counts; otherwise their first slots (k_scan).  kout may be null (the last
// digit of a sort whose caller needs the values only).
template <bool FUSED>
__global__ __launch_bounds__(kSortThreads) void k_scatter(const uint32_t* __restrict__ kin,
                                                          const uint32_t* __restrict__ vin,
                                                          uint32_t* __restrict__ kout, uint32_t* __restrict__ vout,
                                                          const SortTile* __restrict__ tiles,
                                                          const SortSeg* __restrict__ segs,
                                                          const uint32_t* __restrict__ hist, int shift) {
  constexpr int W = kSortThreads / 64;
  static_assert(kSortThreads == 256, "one thread per digit");
  __shared__ uint32_t cnt[W][256];
  __shared__ uint32_t wtot[4];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const SortTile t = tiles[blockIdx.x];
  const SortSeg s = segs[t.seg];
  uint32_t key[kSortItems], val[kSortItems], d[kSortItems], rank[kSortItems];
  bool valid[kSortItems];
#pragma unroll
  for (int r = 0; r < kSortItems; ++r) {
    const int k = w * 64 * kSortItems + 64 * r + lane;
    valid[r] = k < t.count;
    key[r] = valid[r] ? kin[t.start + k] : 0u;
    val[r] = valid[r] ? vin[t.start + k] : 0u;
  }
  uint32_t base;
  if constexpr (FUSED) {
    const int mine = (int)blockIdx.x - s.tile0;
    const uint32_t* h = hist + (int64_t)s.tile0 * 256 + tid;
    uint32_t before = 0, total = 0;
#pragma unroll 8
    for (int k = 0; k < s.n_tiles; ++k) {
      const uint32_t c = h[(int64_t)k * 256];
      before += k < mine ? c : 0u;
      total += c;
    }
    base = digit_exclusive_scan(total, wtot) + before;
  } else {
    base = hist[(int64_t)blockIdx.x * 256 + tid];
  }
#pragma unroll
  for (int r = 0; r < kSortItems; ++r) d[r] = (key[r] >> shift) & 0xffu;
  wave_digit_ranks<kSortItems>(d, valid, cnt[w], rank);
  __syncthreads();
  for (int k = 0; k < W; ++k) {
    const uint32_t c = cnt[k][tid];
    cnt[k][tid] = base;
    base += c;
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kSortItems; ++r)
    if (valid[r]) {
      const uint32_t pos = cnt[w][d[r]] + rank[r];
      if (kout) kout[s.start + pos] = key[r];
      vout[s.start + pos] = val[r];
    }
}

// Places 1 / split of a run of a segment of several: an element's slot is its place in its own run, plus the elements
// of earlier runs up to its key, plus those of later runs below it (runs hold consecutive elements, so that order is
// stable).  Every workgroup reads all keys of the segment into LDS and finds its elements there by binary search, four
// runs' searches in flight.  One workgroup sorting 16,384 elements took 62 us; runs of
// 2,048 and the merge 25, and at 8,192 elements 22 and 17.
constexpr int kMergeThreads = 512;
template <int RUNS>
__global__ __launch_bounds__(kMergeThreads) void k_merge(const uint32_t* __restrict__ keys,
                                                         const uint32_t* __restrict__ vals,
                                                         const SortTile* __restrict__ runs,
                                                         const SortSeg* __restrict__ segs, int split,
                                                         uint32_t* __restrict__ out_keys,
                                                         uint32_t* __restrict__ out_vals) {
  __shared__ uint32_t sh[RUNS * kSortTile];
  const SortTile T = runs[blockIdx.x / split];
  const SortSeg S = segs[T.seg];
  if (T.runs > RUNS || S.count > RUNS * kSortTile) return;  // (uniform; the launch sizes LDS for the largest segment)
  const int t = threadIdx.x;
#pragma unroll 8
  for (int i = t; i < S.count; i += kMergeThreads) sh[i] = keys[S.start + i];
  const int own = (int)((T.start - S.start) / kSortTile);
  const int part = kSortTile / split;
  const int first = (int)(blockIdx.x % split) * part, last = min(T.count, first + part);
  __syncthreads();
  for (int i = first + t; i < last; i += kMergeThreads) {
    const uint32_t key = sh[own * kSortTile + i], val = vals[T.start + i];
    uint32_t slot = (uint32_t)i;
    for (int r0 = 0; r0 < T.runs; r0 += 4) {
      uint32_t pos[4], lim[4];
      int len[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int r = r0 + u;
        pos[u] = 0;
        len[u] = r < T.runs && r != own ? min(kSortTile, S.count - r * kSortTile) : 0;
        lim[u] = key + (r < own ? 1u : 0u);  // (keys are below 2^32 - 1)
      }
#pragma unroll
      for (int step = kSortTile; step > 0; step >>= 1)
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const uint32_t q = pos[u] + (uint32_t)step;
          if ((int)q <= len[u] && sh[(r0 + u) * kSortTile + q - 1] < lim[u]) pos[u] = q;
        }
#pragma unroll
      for (int u = 0; u < 4; ++u) slot += pos[u];
    }
    out_vals[S.start + slot] = val;
    if (out_keys) out_keys[S.start + slot] = key;
  }
}

}  // namespace

hipError_t launch_radix_sort(uint32_t* keys, uint32_t* vals, uint32_t* keys_tmp, uint32_t* vals_tmp, uint32_t* hist,
                             const SortTile* d_tiles, const SortSeg* d_segs, const SortPlan& plan, int bits,
                             bool keep_keys, hipStream_t st) {
  if (plan.n_tiles <= 0) return hipSuccess;
  uint32_t *ki = keys, *vi = vals, *ko = keys_tmp, *vo = vals_tmp;
  for (int shift = 0; shift < bits; shift += 8) {
    uint32_t* kw = shift + 8 < bits || keep_keys ? ko : nullptr;
    if (shift > 0) k_hist<<<plan.n_tiles, kSortThreads, 0, st>>>(ki, d_tiles, shift, hist);
    if (plan.max_seg_tiles <= kFusedTiles) {
      k_scatter<true><<<plan.n_tiles, kSortThreads, 0, st>>>(ki, vi, kw, vo, d_tiles, d_segs, hist, shift);
    } else {
      k_scan<<<plan.n_segs, 256, 0, st>>>(hist, d_segs);
      k_scatter<false><<<plan.n_tiles, kSortThreads, 0, st>>>(ki, vi, kw, vo, d_tiles, d_segs, hist, shift);
    }
    uint32_t* tk = ki; ki = ko; ko = tk;
    uint32_t* tv = vi; vi = vo; vo = tv;
  }
  return hipGetLastError();
}

hipError_t launch_merge(const uint32_t* keys, const uint32_t* vals, const SortTile* d_pieces, const SortSeg* d_segs,
                        const SortPlan& plan, uint32_t* out_keys, uint32_t* out_vals, hipStream_t st) {
  if (plan.n_multi <= 0) return hipSuccess;
  // a few runs take four workgroups each (the chip is empty); many do not read their segments' keys four times
  const int split = plan.n_multi <= 128 ? 4 : 1;
  const unsigned nb = (unsigned)plan.n_multi * split;
  const SortTile* runs = d_pieces + plan.n_tiles;
  if (plan.max_multi <= 4 * kSortTile)
    k_merge<4><<<nb, kMergeThreads, 0, st>>>(keys, vals, runs, d_segs, split, out_keys, out_vals);
  else
    k_merge<8><<<nb, kMergeThreads, 0, st>>>(keys, vals, runs, d_segs, split, out_keys, out_vals);
  static_assert(kMergeMax == 8 * kSortTile, "the largest merge");
  return hipGetLastError();
}

}  // namespace rkhsba

// ---------------------------------------------------------------- exclusive scan (uint32)

namespace rkhsba {
namespace {

constexpr int kScanThreads = 256;
constexpr int kScanItems = 8;
constexpr int kScanTile = kScanThreads * kScanItems;

__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t v, uint32_t* sh, uint32_t* total) {
  const int tid = threadIdx.x;
  sh[tid] = v;
  __syncthreads();
  for (int o = 1; o < kScanThreads; o <<= 1) {
    const uint32_t add = tid >= o ? sh[tid - o] : 0u;
    __syncthreads();
    sh[tid] += add;
    __syncthreads();
  }
  const uint32_t incl = sh[tid];
  if (total) *total = sh[kScanThreads - 1];
  __syncthreads();
  return incl - v;
}

// Per tile: sum of the tile.
__global__ __launch_bounds__(kScanThreads) void k_scan_reduce(const uint32_t* __restrict__ in, int64_t n,
                                                              uint32_t* __restrict__ tile_sums) {
  __shared__ uint32_t sh[kScanThreads];
  const int64_t base = (int64_t)blockIdx.x * kScanTile;
  uint32_t s = 0;
  for (int r = 0; r < kScanItems; ++r) {
    const int64_t i = base + (int64_t)threadIdx.x * kScanItems + r;
    if (i < n) s += in[i];
  }
  uint32_t tot;
  block_exclusive_scan(s, sh, &tot);
  if (threadIdx.x == 0) tile_sums[blockIdx.x] = tot;
}

// Single block: exclusive scan of the tile sums (sequential over chunks of 256).
__global__ __launch_bounds__(kScanThreads) void k_scan_tiles(uint32_t* __restrict__ tile_sums, int n_tiles,
                                                             uint64_t* __restrict__ total) {
  __shared__ uint32_t sh[kScanThreads];
  uint64_t carry = 0;
  for (int c = 0; c < n_tiles; c += kScanThreads) {
    const int i = c + threadIdx.x;
    const uint32_t v = i < n_tiles ? tile_sums[i] : 0u;
    uint32_t tot;
    const uint32_t ex = block_exclusive_scan(v, sh, &tot);
    if (i < n_tiles) tile_sums[i] = (uint32_t)(carry + ex);
    carry += tot;
  }
  if (threadIdx.x == 0 && total) *total = carry;
}

__global__ __launch_bounds__(kScanThreads) void k_scan_apply(const uint32_t* __restrict__ in, int64_t n,
                                                             const uint32_t* __restrict__ tile_sums,
                                                             uint32_t* __restrict__ out) {
  __shared__ uint32_t sh[kScanThreads];
  const int64_t base = (int64_t)blockIdx.x * kScanTile;
  uint32_t v[kScanItems];
  uint32_t s = 0;
  for (int r = 0; r < kScanItems; ++r) {
    const int64_t i = base + (int64_t)threadIdx.x * kScanItems + r;
    v[r] = i < n ? in[i] : 0u;
    s += v[r];
  }
  uint32_t run = block_exclusive_scan(s, sh, nullptr) + tile_sums[blockIdx.x];
  for (int r = 0; r < kScanItems; ++r) {
    const int64_t i = base + (int64_t)threadIdx.x * kScanItems + r;
    if (i < n) out[i] = run;
    run += v[r];
  }
}

}  // namespace

// out[i] = sum_{k<i} in[i] (may alias in); *d_total (device, nullable) = sum of all.
// tmp: at least ceil(n / 2048) uint32.
hipError_t launch_exclusive_scan(const uint32_t* in, uint32_t* out, int64_t n, uint32_t* tmp, uint64_t* d_total,
                                 hipStream_t st) {
  const int64_t tiles = (n + kScanTile - 1) / kScanTile;
  if (tiles > 0) {
    k_scan_reduce<<<(unsigned)tiles, kScanThreads, 0, st>>>(in, n, tmp);
    k_scan_tiles<<<1, kScanThreads, 0, st>>>(tmp, (int)tiles, d_total);
    k_scan_apply<<<(unsigned)tiles, kScanThreads, 0, st>>>(in, n, tmp, out);
  } else if (d_total) {
    hipMemsetAsync(d_total, 0, sizeof(uint64_t), st);
  }
  return hipGetLastError();
}

}  // namespace rkhsba
