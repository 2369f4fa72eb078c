// Voxel-structure build: frame bounds, cell keys, gather into key order, and
// the per-row cell tables used by the candidate sweeps.  Runs once per
// set of frames; each frame is hashed in its own local coordinates, so the
// structure does not depend on the poses.
#include <algorithm>
#include <cfloat>
#include <climits>

#include "block_sort.h"

namespace rkhsba {
namespace {

constexpr int kThreads = 256;

__device__ inline void frame_of(const int64_t* __restrict__ off, int K, int64_t i, int& f, int64_t& local) {
  f = upper_segment(off, K, i);
  local = i - off[f];
}

// The bits of a float as an unsigned integer in the floats' order (float_of_ordered undoes it).
__device__ inline uint32_t ordered_bits(float v) {
  const uint32_t u = __float_as_uint(v);
  return (u & 0x80000000u) ? ~u : u | 0x80000000u;
}

// Smallest and largest coordinate per frame and axis (and, with class ids, the largest id).  floor(x * inv_cell) is
// monotone in x, so these bound the cells of a grid of any cell size, and the keys are computed from the points where
// they are needed: cell coordinates that a first kernel stored cost 24 bytes per point, and a second one for the
// grid of the chosen size.  A block takes chunks of kBoundPoints points of one frame and reads them as consecutive
// floats, thread t those of axis t % 3; its seven words are reduced in LDS and leave in one atomic each.  (Blocks of
// 4,096 points over the concatenated frames took per-point atomics where more than two frames met: 8 frames x 2,000
// points 140 us, now 12.)
// bounds: [f * 6 + 0..2] smallest, [f * 6 + 3..5] largest, as ordered_bits; *bad: a coordinate is not finite.
constexpr int kBoundThreads = 192;
constexpr int kBoundItems = 16;
constexpr int kBoundPoints = kBoundThreads * kBoundItems / 3;
// Points per thread of the row extents: one, except where the blocks' atomics on the one counter would serialise
// (6.4 million points).
constexpr int64_t kExtentFew = 1 << 20;
inline int extent_items(int64_t n) { return n <= kExtentFew ? 1 : 4; }

__global__ __launch_bounds__(kBoundThreads) void k_frame_bounds(const float* const* __restrict__ xyz,
                                                                const int64_t* __restrict__ off, int per_frame,
                                                                const void* const* __restrict__ cls,
                                                                uint32_t* __restrict__ bounds,
                                                                int32_t* __restrict__ bad,
                                                                int32_t* __restrict__ label_max) {
  __shared__ uint32_t sb[6];
  __shared__ int32_t sl;
  const int t = threadIdx.x;
  if (t < 3) {
    sb[t] = 0xffffffffu;
    sb[3 + t] = 0u;
  }
  if (t == 3) sl = -1;
  __syncthreads();
  const int f = blockIdx.x / per_frame;
  const int64_t n = off[f + 1] - off[f];
  const float* __restrict__ p = xyz[f];
  uint32_t mn = 0xffffffffu, mx = 0u;
  int lab = -1;
  bool wrong = false;
  for (int64_t c = blockIdx.x % per_frame; c * kBoundPoints < n; c += per_frame) {
#pragma unroll
    for (int r = 0; r < kBoundItems; ++r) {
      const int64_t j = 3 * c * kBoundPoints + r * kBoundThreads + t;
      if (j < 3 * n) {
        const float v = p[j];
        wrong = wrong || !(fabsf(v) <= FLT_MAX);
        const uint32_t o = ordered_bits(v);
        mn = min(mn, o);
        mx = max(mx, o);
      }
    }
    if (label_max) {
      const uint16_t* __restrict__ id = static_cast<const uint16_t*>(cls[f]);
      for (int k = t; k < kBoundPoints; k += kBoundThreads)
        if (c * kBoundPoints + k < n) lab = max(lab, (int)id[c * kBoundPoints + k]);
    }
  }
  atomicMin(&sb[t % 3], mn);
  atomicMax(&sb[3 + t % 3], mx);
  if (label_max) atomicMax(&sl, lab);
  if (__ballot(wrong) && wrong) atomicOr(bad, 1);
  __syncthreads();
  if (t < 3 && sb[t] != 0xffffffffu) atomicMin(&bounds[6 * f + t], sb[t]);
  else if (t >= 3 && t < 6 && sb[t] != 0u) atomicMax(&bounds[6 * f + t], sb[t]);
  else if (t == 6 && label_max && sl >= 0) atomicMax(&label_max[f], sl);
}

// Cell key of point l of frame F; in a label-stacked frame the class id selects the layer of NZ cells that the
// point's z cell lies in (kz' = id * NZ + kz).  k = floor(x * inv_cell) per axis in FP64.
__device__ inline uint32_t cell_key(const float* const* __restrict__ xyz, double inv_cell, const FrameInfo& F,
                                    const void* const* __restrict__ cls, int f, int64_t l) {
  const float* c = xyz[f] + 3 * l;
  const uint32_t kx = (uint32_t)((int)floor((double)c[0] * inv_cell) - F.org[0]);
  const uint32_t ky = (uint32_t)((int)floor((double)c[1] * inv_cell) - F.org[1]);
  uint32_t kz = (uint32_t)((int)floor((double)c[2] * inv_cell) - F.org[2]);
  if (F.n_lab > 0) kz += (uint32_t)static_cast<const uint16_t*>(cls[f])[l] * (uint32_t)F.dim[2];
  return (kz * (uint32_t)F.dim[1] + ky) * (uint32_t)F.dim[0] + kx;
}

// One block per sort tile of a frame: keys, point indices and the tile's histogram of the first digit.
__global__ __launch_bounds__(kSortThreads) void k_cell_keys(const float* const* __restrict__ xyz, double inv_cell,
                                                            const FrameInfo* __restrict__ frames,
                                                            const void* const* __restrict__ cls,
                                                            const SortTile* __restrict__ tiles,
                                                            uint32_t* __restrict__ keys, uint32_t* __restrict__ vals,
                                                            uint32_t* __restrict__ hist) {
  __shared__ uint32_t h[256];
  static_assert(kSortThreads == 256, "one thread per digit");
  h[threadIdx.x] = 0u;
  __syncthreads();
  const SortTile t = tiles[blockIdx.x];
  const FrameInfo F = frames[t.edge];
  for (int k = threadIdx.x; k < t.count; k += kSortThreads) {
    const int64_t i = t.start + k, l = i - F.pt_off;
    const uint32_t key = cell_key(xyz, inv_cell, F, cls, t.edge, l);
    keys[i] = key;
    vals[i] = (uint32_t)l;
    atomicAdd(&h[key & 0xffu], 1u);
  }
  __syncthreads();
  hist[(int64_t)blockIdx.x * 256 + threadIdx.x] = h[threadIdx.x];
}

// One workgroup per run: keys, and their sort in LDS; the only run of its frame is done, the others are merged.
constexpr int kRunThreads = 512, kRunItems = 4;
__global__ __launch_bounds__(kRunThreads) void k_cell_runs(const float* const* __restrict__ xyz, double inv_cell,
                                                           const FrameInfo* __restrict__ frames,
                                                           const void* const* __restrict__ cls,
                                                           const SortTile* __restrict__ runs, int bits,
                                                           uint32_t* __restrict__ run_keys,
                                                           uint32_t* __restrict__ run_vals,
                                                           uint32_t* __restrict__ sorted_keys,
                                                           uint32_t* __restrict__ sorted_vals) {
  static_assert(kRunThreads * kRunItems == kSortTile, "a run");
  __shared__ typename BlockSort<kRunThreads, kRunItems>::Shared sh;
  const SortTile T = runs[blockIdx.x];
  const FrameInfo F = frames[T.edge];
  const int64_t first = T.start - F.pt_off;
  const int base = (int)(threadIdx.x >> 6) * 64 * kRunItems + (int)(threadIdx.x & 63);
  uint32_t key[kRunItems];
#pragma unroll
  for (int r = 0; r < kRunItems; ++r)
    key[r] = base + 64 * r < T.count ? cell_key(xyz, inv_cell, F, cls, T.edge, first + base + 64 * r) : 0u;
  BlockSort<kRunThreads, kRunItems>::sort(key, T.count, bits, sh);
  uint32_t* __restrict__ keys = T.runs == 1 ? sorted_keys : run_keys;
  uint32_t* __restrict__ vals = T.runs == 1 ? sorted_vals : run_vals;
  for (int i = threadIdx.x; i < T.count; i += kRunThreads) {
    keys[T.start + i] = sh.key[i];
    vals[T.start + i] = (uint32_t)first + sh.val[i];
  }
}

// One block per frame: the first point (frame-local sorted index) of each
// label layer of a label-stacked frame, by binary search over its sorted keys.
__global__ __launch_bounds__(kThreads) void k_label_starts(const uint32_t* __restrict__ keys,
                                                           const FrameInfo* __restrict__ frames,
                                                           const int64_t* __restrict__ lab_off,
                                                           int32_t* __restrict__ out) {
  const FrameInfo F = frames[blockIdx.x];
  if (F.n_lab <= 0) return;
  const uint32_t* k = keys + F.pt_off;
  const uint64_t layer = (uint64_t)F.dim[0] * F.dim[1] * F.dim[2];
  for (int L = threadIdx.x; L <= F.n_lab; L += kThreads) {
    const uint64_t first = (uint64_t)L * layer;  // smallest key of layer L
    int lo = 0, hi = F.n;                        // first index with key >= first
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if ((uint64_t)k[mid] < first) lo = mid + 1; else hi = mid;
    }
    out[lab_off[blockIdx.x] + L] = lo;
  }
}

// Round to nearest even: float32 -> bfloat16 (finite inputs).
__device__ inline uint16_t f32_to_bf16(float v) {
  const uint32_t u = __float_as_uint(v);
  return (uint16_t)((u + 0x7fffu + ((u >> 16) & 1u)) >> 16);
}

// Round to nearest even: float32 -> OCP fp8 e4m3 (bias 7, 3 mantissa bits,
// subnormal step 2^-9), saturating at the largest finite value 448.
__device__ inline uint8_t f32_to_e4m3(float v) {
  const uint32_t u = __float_as_uint(v);
  const uint32_t sign = (u >> 24) & 0x80u;
  const uint32_t a = u & 0x7fffffffu;
  uint32_t code;
  if (a >= 0x43e00000u) {          // |v| >= 448
    code = 0x7eu;
  } else if (a < 0x3c800000u) {    // |v| < 2^-6: multiples of 2^-9
    code = (uint32_t)rintf(__uint_as_float(a) * 512.0f);  // 0..8; 8 is the smallest normal, 2^-6
  } else {
    const uint32_t r = (a + 0x7ffffu + ((a >> 20) & 1u)) >> 20;  // biased exponent and 3 mantissa bits, rounded
    code = r - (120u << 3);                                       // exponent bias 127 -> 7
    if (code > 0x7eu) code = 0x7eu;
  }
  return (uint8_t)(sign | code);
}

// Gathers points into key order.  pts.w carries the class id bits for one-hot
// features.
__global__ __launch_bounds__(kThreads) void k_gather(const float* const* __restrict__ xyz,
                                                     const void* const* __restrict__ feats, int feat_kind,
                                                     const int64_t* __restrict__ off, int K, int64_t n_total,
                                                     const uint32_t* __restrict__ sorted_keys,
                                                     const uint32_t* __restrict__ sorted_vals,
                                                     float4* __restrict__ pts, int32_t* __restrict__ perm,
                                                     uint32_t* __restrict__ keys) {
  const int64_t p = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (p >= n_total) return;
  int f;
  int64_t s;
  frame_of(off, K, p, f, s);
  const int64_t o = sorted_vals[p];
  const float* x = xyz[f] + 3 * o;
  float w = 0.0f;
  if (feat_kind == 0) w = __uint_as_float((uint32_t)((const uint16_t*)feats[f])[o]);
  pts[p] = make_float4(x[0], x[1], x[2], w);
  perm[p] = (int32_t)o;
  keys[p] = sorted_keys[p];
}

// Gathers dense feature rows into key order, stored in the feature path's
// element type and zero padded to Dp.  One thread per stored element, in
// storage order: consecutive threads read consecutive elements of a point's
// input row and write consecutive stored elements (one thread per point would
// touch 64 scattered rows with every load and store).  IDX: the element index
// type (32 bits whenever n_total * Dp fits).
template <typename IDX>
__global__ __launch_bounds__(kThreads) void k_gather_feat(const void* const* __restrict__ feats, int feat_kind, int D,
                                                          int Dp, const int64_t* __restrict__ off, int K,
                                                          int64_t n_total, const uint32_t* __restrict__ sorted_vals,
                                                          void* __restrict__ feat, int32_t* __restrict__ neg_flag) {
  const IDX i = (IDX)blockIdx.x * kThreads + threadIdx.x;
  bool neg = false;
  if ((int64_t)i < n_total * Dp) {
    const IDX p = i / (IDX)Dp;
    const int k = (int)(i - p * (IDX)Dp);
    int f;
    int64_t s;
    frame_of(off, K, (int64_t)p, f, s);
    const int64_t o = sorted_vals[p];
    const float v = k < D ? static_cast<const float*>(feats[f])[o * D + k] : 0.0f;
    neg = v < 0.0f;
    if (feat_kind == 1) static_cast<float*>(feat)[p * (IDX)Dp + (IDX)feat_slot(1, Dp, k)] = v;
    else if (feat_kind == 2) static_cast<uint16_t*>(feat)[i] = f32_to_bf16(v);
    else static_cast<uint8_t*>(feat)[i] = f32_to_e4m3(v);
  }
  // some inner products may be negative: one atomic per wavefront with such an element, none once the flag is
  // set (a per-element atomic on the one flag word serialises)
  const unsigned long long negs = __ballot(neg);
  if (negs && (int)(threadIdx.x & 63) == __builtin_ctzll(negs) && __atomic_load_n(neg_flag, __ATOMIC_RELAXED) == 0)
    atomicOr(neg_flag, 1);
}

__device__ inline void decode(uint32_t key, const FrameInfo& F, int& kx, int& ky, int& kz) {
  const uint32_t nx = (uint32_t)F.dim[0], ny = (uint32_t)F.dim[1];
  kx = (int)(key % nx);
  const uint32_t r = key / nx;
  ky = (int)(r % ny);
  kz = (int)(r / ny);
}

// Smallest value of each feature dimension over n rows of Dp FP32 values: the
// block size and the grid stride are multiples of Dp, so every thread sees
// one dimension (threadIdx.x % Dp) and reads the rows' values coalesced.
// out[d] (bit patterns of non-negative floats, ordered as integers) must hold
// +inf or a larger earlier minimum; negative values count as 0.
__global__ __launch_bounds__(kThreads) void k_feature_min(const float* __restrict__ feat, int64_t total, int Dp,
                                                          uint32_t* __restrict__ out) {
  __shared__ uint32_t sm[64];
  const int t = threadIdx.x;
  if (t < Dp) sm[t] = 0x7f800000u;
  __syncthreads();
  float m = FLT_MAX;
#pragma unroll 8
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + t; e < total; e += (int64_t)gridDim.x * blockDim.x)
    m = fminf(m, feat[e]);
  atomicMin(&sm[t % Dp], __float_as_uint(fmaxf(m, 0.0f)));
  __syncthreads();
  if (t < Dp) atomicMin(&out[t], sm[t]);
}

__global__ __launch_bounds__(kThreads) void k_row_init(int4* __restrict__ rows, int64_t n_rows,
                                                       uint64_t* __restrict__ totals) {
  const int64_t r = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (r < n_rows) rows[r] = make_int4(INT_MAX, INT_MIN, 0, 0);
  if (r < 2) totals[r] = 0;
}

// The x extent of every occupied row: a frame's points are sorted by key, so
// the points of one row are contiguous, and its first and last points give
// x_lo and x_hi (plain stores, no atomics).  Counts the occupied cells, with
// one atomic per block on the single counter.
__global__ __launch_bounds__(kThreads) void k_row_extent(const uint32_t* __restrict__ keys,
                                                         const FrameInfo* __restrict__ frames,
                                                         const int64_t* __restrict__ off, int K, int64_t n_total,
                                                         int4* __restrict__ rows, uint64_t* __restrict__ n_cells,
                                                         int items) {
  __shared__ uint32_t heads_sh;
  if (threadIdx.x == 0) heads_sh = 0u;
  __syncthreads();
  uint32_t heads = 0;
  for (int it = 0; it < items; ++it) {
    const int64_t p = ((int64_t)blockIdx.x * items + it) * kThreads + threadIdx.x;
    if (p >= n_total) break;
    int f;
    int64_t s;
    frame_of(off, K, p, f, s);
    const FrameInfo& F = frames[f];
    const uint32_t nx = (uint32_t)F.dim[0];
    const uint32_t key = keys[p], prev = s == 0 ? ~key : keys[p - 1];
    const uint32_t row = key / nx;
    const bool head = s == 0 || prev / nx != row;
    const bool tail = s + 1 == F.n || keys[p + 1] / nx != row;
    int4* R = rows + F.row_off + (int64_t)row;
    if (head) R->x = (int)(key - row * nx);
    if (tail) R->y = (int)(key - row * nx);
    heads += prev != key ? 1u : 0u;
  }
  heads = wave_inclusive_scan(heads);
  if ((threadIdx.x & 63) == 63) atomicAdd(&heads_sh, heads);
  __syncthreads();
  if (threadIdx.x == 0 && heads_sh) atomicAdd((unsigned long long*)n_cells, (unsigned long long)heads_sh);
}

// A row table of up to kRowBlockMax rows in one workgroup: the entries of the rows before each (a scan of their
// sizes, 1,024 rows a step): 5 us for 8,192 rows, 22 us for 32,768, where the five launches of the general scan take
// 20 with the gaps between them.
constexpr int kRowBlockMax = 32768;
__global__ __launch_bounds__(1024) void k_row_offsets(int4* __restrict__ rows, int n_rows,
                                                      uint64_t* __restrict__ total) {
  __shared__ uint32_t wt[2][16];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  constexpr int B = 8;
  uint64_t carry = 0;
  for (int base = 0; base < n_rows; base += B * 1024) {
    uint32_t size[B];
#pragma unroll
    for (int r = 0; r < B; ++r) {
      const int i = base + r * 1024 + t;
      const int2 x = i < n_rows ? *reinterpret_cast<const int2*>(rows + i) : make_int2(INT_MAX, INT_MIN);
      size[r] = x.y >= x.x ? (uint32_t)(x.y - x.x + 2) : 0u;
    }
#pragma unroll
    for (int r = 0; r < B; ++r) {
      const uint32_t incl = wave_inclusive_scan(size[r]);
      if (lane == 63) wt[r & 1][w] = incl;
      __syncthreads();
      uint64_t before = 0, all = 0;
#pragma unroll
      for (int k = 0; k < 16; ++k) {
        const uint32_t v = wt[r & 1][k];
        before += k < w ? v : 0u;
        all += v;
      }
      const int i = base + r * 1024 + t;
      if (i < n_rows) rows[i].z = (int)(uint32_t)(carry + before + incl - size[r]);
      carry += all;
    }
  }
  if (t == 0) *total = carry;
}

__global__ __launch_bounds__(kThreads) void k_row_sizes(const int4* __restrict__ rows, int64_t n_rows,
                                                        uint32_t* __restrict__ sizes) {
  const int64_t r = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (r >= n_rows) return;
  const int4 v = rows[r];
  sizes[r] = v.y >= v.x ? (uint32_t)(v.y - v.x + 2) : 0u;
}

__global__ __launch_bounds__(kThreads) void k_row_store_offsets(const uint32_t* __restrict__ offs, int64_t n_rows,
                                                                int4* __restrict__ rows) {
  const int64_t r = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (r < n_rows) rows[r].z = (int)offs[r];
}

// xtab[row][x - x_lo] = first point (frame-local sorted index) of cell x or,
// for an empty cell, of the next occupied cell in the row; the entry after
// x_hi is the end of the row.  Every entry is written by exactly one thread:
// the head of each occupied cell fills the entries from the previous occupied
// cell of the row (exclusive) up to its own; the row's last point writes the
// end entry.
__global__ __launch_bounds__(kThreads) void k_xtab_fill(const uint32_t* __restrict__ keys,
                                                        const FrameInfo* __restrict__ frames,
                                                        const int64_t* __restrict__ off, int K, int64_t n_total,
                                                        const int4* __restrict__ rows, uint32_t* __restrict__ xtab) {
  const int64_t p = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (p >= n_total) return;
  int f;
  int64_t s;
  frame_of(off, K, p, f, s);
  const FrameInfo& F = frames[f];
  const uint32_t key = keys[p];
  int kx, ky, kz;
  decode(key, F, kx, ky, kz);
  const int64_t row = (int64_t)kz * F.dim[1] + ky;
  const int4 R = rows[F.row_off + row];
  uint32_t* xt = xtab + F.xt_off + (uint32_t)R.z;
  const bool has_prev = s > 0;
  const bool has_next = s + 1 < F.n;
  const uint32_t kprev = has_prev ? keys[p - 1] : 0u;
  const bool head = !has_prev || kprev != key;
  if (head) {  // head of an occupied cell
    int x0 = R.x;
    if (has_prev) {
      int px, py, pz;
      decode(kprev, F, px, py, pz);
      if ((int64_t)pz * F.dim[1] + py == row) x0 = px + 1;
    }
    for (int x = x0; x <= kx; ++x) xt[x - R.x] = (uint32_t)s;
  }
  bool row_end = !has_next;
  if (has_next) {
    int nx, ny, nz;
    decode(keys[p + 1], F, nx, ny, nz);
    row_end = (int64_t)nz * F.dim[1] + ny != row;
  }
  if (row_end) xt[R.y + 1 - R.x] = (uint32_t)(s + 1);
}

// Centroid of one frame: each thread sums a strided subset in FP64, then the
// partial sums are added in thread order.
__global__ __launch_bounds__(kThreads) void k_frame_centroid(const float4* __restrict__ pts, int n,
                                                             double* __restrict__ out) {
  __shared__ double sh[3][kThreads];
  double s[3] = {0.0, 0.0, 0.0};
  for (int i = threadIdx.x; i < n; i += kThreads) {
    const float4 p = pts[i];
    s[0] += p.x;
    s[1] += p.y;
    s[2] += p.z;
  }
  for (int a = 0; a < 3; ++a) sh[a][threadIdx.x] = s[a];
  __syncthreads();
  if (threadIdx.x < 3) {
    double t = 0.0;
    for (int k = 0; k < kThreads; ++k) t += sh[threadIdx.x][k];
    out[threadIdx.x] = n > 0 ? t / n : 0.0;
  }
}

inline unsigned blocks(int64_t n) { return (unsigned)((n + kThreads - 1) / kThreads); }

}  // namespace

hipError_t launch_frame_centroid(const float4* d_pts, int n, double* d_out, hipStream_t st) {
  k_frame_centroid<<<1, kThreads, 0, st>>>(d_pts, n, d_out);
  return hipGetLastError();
}

hipError_t launch_frame_bounds(const float* const* d_xyz_ptrs, const int64_t* d_in_off, int K, int64_t n_max,
                               const void* const* d_class_ptrs, uint32_t* d_bounds, int32_t* d_bad,
                               int32_t* d_label_max, hipStream_t st) {
  if (K <= 0 || (d_label_max && !d_class_ptrs)) return hipErrorInvalidValue;
  // blocks per frame: a chunk each while they fill the chip, and no fewer than 64 (frames of unequal sizes)
  const int64_t chunks = (n_max + kBoundPoints - 1) / kBoundPoints;
  const int per_frame = (int)std::max<int64_t>(1, std::min<int64_t>(chunks, std::max(64, 8192 / K)));
  k_frame_bounds<<<(unsigned)K * per_frame, kBoundThreads, 0, st>>>(d_xyz_ptrs, d_in_off, per_frame, d_class_ptrs,
                                                                    d_bounds, d_bad, d_label_max);
  return hipGetLastError();
}

hipError_t launch_cell_sort(const float* const* d_xyz_ptrs, double inv_cell, const FrameInfo* d_frames,
                            const void* const* d_class_ptrs, const SortTile* d_tiles, const SortSeg* d_segs,
                            const SortPlan& plan, int bits, uint32_t* d_keys, uint32_t* d_vals, uint32_t* d_hist,
                            uint32_t* d_run_keys, uint32_t* d_run_vals, uint32_t* d_sorted_keys,
                            uint32_t* d_sorted_vals, hipStream_t st) {
  if (plan.n_tiles > 0)
    k_cell_keys<<<(unsigned)plan.n_tiles, kSortThreads, 0, st>>>(d_xyz_ptrs, inv_cell, d_frames, d_class_ptrs,
                                                                 d_tiles, d_keys, d_vals, d_hist);
  if (plan.n_runs > 0)
    k_cell_runs<<<(unsigned)plan.n_runs, kRunThreads, 0, st>>>(d_xyz_ptrs, inv_cell, d_frames, d_class_ptrs,
                                                               d_tiles + plan.n_tiles, bits, d_run_keys, d_run_vals,
                                                               d_sorted_keys, d_sorted_vals);
  hipError_t e = launch_merge(d_run_keys, d_run_vals, d_tiles, d_segs, plan, d_sorted_keys, d_sorted_vals, st);
  if (e != hipSuccess) return e;
  return hipGetLastError();
}

hipError_t launch_label_starts(const uint32_t* d_keys, const FrameInfo* d_frames, const int64_t* d_lab_off, int K,
                               int32_t* d_out, hipStream_t st) {
  if (K > 0) k_label_starts<<<K, kThreads, 0, st>>>(d_keys, d_frames, d_lab_off, d_out);
  return hipGetLastError();
}

hipError_t launch_gather(const float* const* d_xyz_ptrs, const void* const* d_feat_ptrs, int feat_kind, int D, int Dp,
                         const int64_t* d_in_off, int K, int64_t n_total, const uint32_t* d_sorted_keys,
                         const uint32_t* d_sorted_vals, float4* d_pts, void* d_feat, int32_t* d_perm,
                         uint32_t* d_keys, int32_t* d_neg_flag, hipStream_t st) {
  if (n_total <= 0) return hipSuccess;
  k_gather<<<blocks(n_total), kThreads, 0, st>>>(d_xyz_ptrs, d_feat_ptrs, feat_kind, d_in_off, K, n_total,
                                                 d_sorted_keys, d_sorted_vals, d_pts, d_perm, d_keys);
  if (feat_kind != 0) {
    const int64_t total = n_total * Dp;
    if (total <= (int64_t)UINT32_MAX - kThreads)
      k_gather_feat<uint32_t><<<blocks(total), kThreads, 0, st>>>(d_feat_ptrs, feat_kind, D, Dp, d_in_off, K, n_total,
                                                                  d_sorted_vals, d_feat, d_neg_flag);
    else
      k_gather_feat<uint64_t><<<blocks(total), kThreads, 0, st>>>(d_feat_ptrs, feat_kind, D, Dp, d_in_off, K, n_total,
                                                                  d_sorted_vals, d_feat, d_neg_flag);
  }
  return hipGetLastError();
}

hipError_t launch_feature_min(const float* d_feat, int64_t n, int Dp, uint32_t* d_min, hipStream_t st) {
  if (Dp <= 0 || Dp > 64 || n <= 0) return Dp > 64 ? hipErrorInvalidValue : hipSuccess;
  const int threads = Dp * (kThreads / Dp);
  const int64_t total = n * Dp;
  // several rows per thread: every block ends in Dp atomics on the same Dp words (1,024 blocks for 16,000 x 24
  // values spent 10 of 11 us on them)
  const unsigned blocks = (unsigned)std::max<int64_t>(1, std::min<int64_t>(1024, total / (16 * threads)));
  k_feature_min<<<blocks, threads, 0, st>>>(d_feat, total, Dp, d_min);
  return hipGetLastError();
}

hipError_t launch_rows(const uint32_t* d_keys, const FrameInfo* d_frames, const int64_t* d_in_off, int K,
                       int64_t n_total, int4* d_rows, int64_t n_rows, uint32_t* d_sizes, uint32_t* d_scan_tmp,
                       uint64_t* d_totals, hipStream_t st) {
  if (n_rows <= 0 || n_total <= 0) return hipErrorInvalidValue;
  k_row_init<<<blocks(n_rows + 1), kThreads, 0, st>>>(d_rows, n_rows, d_totals);
  const int items = extent_items(n_total);
  k_row_extent<<<blocks((n_total + items - 1) / items), kThreads, 0, st>>>(d_keys, d_frames, d_in_off, K, n_total,
                                                                           d_rows, d_totals + 1, items);
  if (n_rows <= kRowBlockMax) {
    k_row_offsets<<<1, 1024, 0, st>>>(d_rows, (int)n_rows, d_totals);
    return hipGetLastError();
  }
  k_row_sizes<<<blocks(n_rows), kThreads, 0, st>>>(d_rows, n_rows, d_sizes);
  hipError_t e = launch_exclusive_scan(d_sizes, d_sizes, n_rows, d_scan_tmp, d_totals, st);
  if (e != hipSuccess) return e;
  k_row_store_offsets<<<blocks(n_rows), kThreads, 0, st>>>(d_sizes, n_rows, d_rows);
  return hipGetLastError();
}

hipError_t launch_xtab(const uint32_t* d_keys, const FrameInfo* d_frames, const int64_t* d_in_off, int K,
                       int64_t n_total, const int4* d_rows, uint32_t* d_xtab, hipStream_t st) {
  if (n_total > 0)
    k_xtab_fill<<<blocks(n_total), kThreads, 0, st>>>(d_keys, d_frames, d_in_off, K, n_total, d_rows, d_xtab);
  return hipGetLastError();
}

}  // namespace rkhsba
